// sq_gemm: the two integer products of the SQ-format linear layer (Section 3.3) on the INT8
// matrix cores of gfx950, with the dequantising epilogue fused.
//
// CDNA4 has no INT4 matrix instruction, so both products run on v_mfma_i32_32x32x32_i8.
// INT4 codes stay packed (two per byte) from HBM through LDS and are widened in registers just
// before the matrix instruction, without sign extension: a nibble placed in the HIGH four bits
// of a byte is the signed byte 16*code, so for a dword p of eight codes
//     (p << 4) & 0xF0F0F0F0   are codes 0,2,4,6 (times 16)      p & 0xF0F0F0F0   are codes 1,3,5,7
// and the accumulators come out as exact multiples (256x when both operands are widened this
// way, 16x when only the weights are), shifted back in the epilogue.  Integer addition is
// order-independent, so the products are bit-exact whatever the K order, as long as both operands
// use the same one.  The order used: a 16-byte chunk of packed codes (32 channels) feeds two
// consecutive matrix instructions; instruction s (0/1) takes dwords 2s, 2s+1 of the chunk as
// [evens of dword 2s | odds of dword 2s | evens of dword 2s+1 | odds of dword 2s+1].  The INT8
// image of the high part is stored in exactly that byte order (see sq_act::hi_dense).
//
// Work split (the large tile): a workgroup of 8 waves computes 128 tokens x 256 output channels; a wave computes
// 64 tokens x 64 channels for BOTH products (2 x 2x2 tiles of 32x32, 128 accumulator registers), so that two waves share
// a SIMD.  That is what the matrix pipe needs: from a single wave v_mfma_i32_32x32x32_i8 issues every 21 ns, whatever
// stands between the instructions, from two waves every 14.5 ns (measured, registers only), and up to six vector
// instructions per matrix instruction are free then.  With 4 waves of 64 x 128 (256 accumulator registers, one wave per
// SIMD, a quarter less LDS traffic per matrix instruction) [4096,4096] x [22016,4096] took 575 us against 526 us,
// [2048,4096] x [12288,4096] 155 against 147 us, the single-product 256 x 256 tile 308 against 275 us.
// Smaller tiles, of which a shape has at most a round, run two groups of four waves per workgroup, each on every other
// K step; where K is short, one group of four waves and several workgroups per compute unit (pick_variant).
// A K step of 128 channels is copied into one of three LDS stages by LDS-direct loads, two steps
// ahead of its use.  LDS rows are row-major with the 16-byte chunk index XOR-swizzled by the row,
// which keeps the operand reads (32 consecutive rows per half wave) free of bank conflicts.
#include "sq_gemm_common.h"

namespace sq {
namespace {

using namespace gemm;

constexpr int KS = 128;  // channels per K step
constexpr int kHugeMinTiles = 512;  // 256x256 tiles a single-product shape needs to use them

// WITH_LO = false: a tile for loops without a packed low operand (the single-product modes), whose stage
// holds no room for one; that is what lets 256 tokens x 256 channels fit three stages into LDS.
// NS: LDS stages of the K loop.  The copy of step kt + NS - 1 is enqueued while step kt is multiplied, so a copy
// has NS - 2 whole K steps to land before anything waits for it.
template <int BM_, int BN_, int NWM_, int NWN_, bool WITH_LO = true, int S_ = 1, int NS_ = 3>
struct Tile {
  static constexpr int NWM = NWM_, NWN = NWN_;  // waves of a K group: NWM along the tokens, NWN along the channels
  static constexpr int NT = 64 * NWM * NWN;   // threads of a K group
  static constexpr int S = S_;                // K groups; group s takes the K steps s, s + S, ...
  static constexpr int NS = NS_;
  static constexpr int BM = BM_;              // tokens per workgroup
  static constexpr int BN = BN_;              // output channels per workgroup
  static constexpr int WM = BM / NWM;         // tokens per wave
  static constexpr int WN = BN / NWN;         // channels per wave
  static constexpr int TI = WM / 32;          // 32-row tiles per wave along M
  static constexpr int TJ = WN / 32;          // along N
  static constexpr int A_LO = 0;              // [BM][64 B]   packed INT4
  static constexpr int A_HI = WITH_LO ? BM * 64 : 0;  // [BM][128 B]  INT8
  static constexpr int B_OFF = A_HI + BM * 128;  // [BN][64 B] packed INT4
  static constexpr int STAGE = B_OFF + BN * 64;
  static constexpr int LDS_BYTES = S * NS * STAGE;
  static constexpr int THREADS = NT * S;
  static_assert((!WITH_LO || BM * 4 % NT == 0) && BM * 8 % NT == 0 && BN * 4 % NT == 0, "whole copies per wave");
  static_assert(NS >= 3 && LDS_BYTES <= 160 * 1024, "stages must fit in the 160 KB of LDS");
  static_assert((S - 1) * BM * BN * 8 <= LDS_BYTES, "the other groups' partial sums must fit, too");
};

// s_waitcnt immediate (gfx9 encoding: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt_hi[15:14]):
// at most n vector-memory operations (here: LDS-direct loads) outstanding, and no LDS operation.
constexpr int waitcnt_vm_lgkm0(int n) { return (n & 15) | (7 << 4) | (0 << 8) | ((n >> 4) << 14); }

// Workgroup barrier for the K loop.  __syncthreads() would also wait for every outstanding
// LDS-direct load (its release fence drains vmcnt), i.e. for the copy that was enqueued a moment
// ago for two steps ahead.  Here the wave waits only until at most `pending` of its loads are in
// flight (loads retire in order, so the older step is complete) and until its own LDS reads have
// returned, then joins the barrier.  The empty asm statements stop the compiler from moving
// memory accesses across it.
template <int PENDING>
__device__ __forceinline__ void pipeline_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(PENDING));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Operand sources of one K loop and the asynchronous copy of one K step into an LDS stage.
// LO: the packed low part is an operand; HI: an INT8 operand (the zero-padded image of the high
// part, or the compact high codes) is.  The copy uses LDS-direct loads (global_load_lds_dwordx4):
// each wave instruction moves 64 x 16 bytes into 1 KB of LDS, lane l landing at byte 16*l, so the
// XOR swizzle is applied on the global side: the lane that lands in position p of a row fetches
// chunk p ^ swizzle(row).  Four (or eight) consecutive lanes still read 64 (128) contiguous bytes.
template <typename T, bool LO, bool HI>
struct Pipe {
  static constexpr int N_LO = LO ? T::BM * 4 / T::NT : 0;
  static constexpr int N_HI = HI ? T::BM * 8 / T::NT : 0;
  static constexpr int N_B = T::BN * 4 / T::NT;
  static constexpr int NLOAD = N_LO + N_HI + N_B;  // loads per wave per K step

  const char* p_lo[N_LO > 0 ? N_LO : 1];  // per-lane source of each load at k = 0
  const char* p_hi[N_HI > 0 ? N_HI : 1];
  const char* p_b[N_B];
  int kc_lo, kc_hi;  // first channel of this lane's chunk inside a K step (packed operands / INT8 operand)
  int kext;          // channels in this loop (multiple of 32)
  int wave;          // uniform, inside the K group
  int grp;           // K group (uniform)
  int steps;         // K steps of a group
  int rot;           // step the loop starts with (the steps then wrap around)

  __device__ __forceinline__ void init(const uint8_t* a_lo, int64_t lda_lo, const int8_t* a_hi, int64_t lda_hi,
                                       const uint8_t* b, int64_t ldb, int kext_, int m0, int n0, int M, int N, int rot8) {
    const int tid = threadIdx.x & (T::NT - 1);
    kext = kext_;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    grp = T::S == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / T::NT);
    steps = (kext + KS * T::S - 1) / (KS * T::S);
    // With two K groups (few tiles: operands come from far, little is shared) every XCD starts at its own place of K, so
    // that rows 4 KB apart are not asked for at the same few hundred bytes by the whole chip at a time.  Only the last
    // step may be partial (see issue), so the order is turned only where no step is.
    rot = T::S > 1 && kext % (KS * T::S) == 0 ? rot8 * steps / 8 : 0;
    {
      const int row = tid >> 2;  // rows of later loads differ by a multiple of 64: same swizzle
      kc_lo = (((tid & 3) ^ (row >> 2)) & 3) * 32;
    }
    {
      const int row = tid >> 3;  // rows of later loads differ by a multiple of 32
      kc_hi = (((tid & 7) ^ (row >> 1)) & 7) * 16;
    }
#pragma unroll
    for (int i = 0; i < N_LO; ++i) {
      const int m = min(m0 + ((tid + T::NT * i) >> 2), M - 1);
      p_lo[i] = reinterpret_cast<const char*>(a_lo) + m * lda_lo + (kc_lo >> 1);
    }
#pragma unroll
    for (int i = 0; i < N_HI; ++i) {
      const int m = min(m0 + ((tid + T::NT * i) >> 3), M - 1);
      p_hi[i] = reinterpret_cast<const char*>(a_hi) + m * lda_hi + kc_hi;
    }
#pragma unroll
    for (int i = 0; i < N_B; ++i) {
      const int n = min(n0 + ((tid + T::NT * i) >> 2), N - 1);
      p_b[i] = reinterpret_cast<const char*>(b) + n * ldb + (kc_lo >> 1);
    }
  }

  // Enqueue the copy of K step `step` into `stage`.  TAIL: the step may reach past kext (only the last
  // step of a loop can); its chunks past the end come from kZeroChunk.
  template <bool TAIL>
  __device__ __forceinline__ void issue(char* stage, int step) const {
    int turned = step;
    if constexpr (T::S > 1) {
      turned += rot;
      turned = turned >= steps ? turned - steps : turned;
    }
    const int k0 = (turned * T::S + grp) * KS;
    const char* zero = reinterpret_cast<const char*>(kZeroChunk);
    const bool lo_ok = !TAIL || (k0 + kc_lo < kext);
    const bool hi_ok = !TAIL || (k0 + kc_hi < kext);
#pragma unroll
    for (int i = 0; i < N_LO; ++i) {
      const char* src = lo_ok ? p_lo[i] + (k0 >> 1) : zero;
      __builtin_amdgcn_global_load_lds(src, (lds_ptr_t)(stage + T::A_LO + (T::NT * i + 64 * wave) * 16), 16, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < N_HI; ++i) {
      const char* src = hi_ok ? p_hi[i] + k0 : zero;
      __builtin_amdgcn_global_load_lds(src, (lds_ptr_t)(stage + T::A_HI + (T::NT * i + 64 * wave) * 16), 16, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < N_B; ++i) {
      const char* src = lo_ok ? p_b[i] + (k0 >> 1) : zero;
      __builtin_amdgcn_global_load_lds(src, (lds_ptr_t)(stage + T::B_OFF + (T::NT * i + 64 * wave) * 16), 16, 0, 0);
    }
  }
};

// The operands one wave needs for 64 channels (two matrix instructions deep) of its tile.
template <typename T>
struct Frags {
  v4u alo[T::TI];     // packed low codes: 32 channels per row tile
  v4u bw[T::TJ];      // packed weight codes
  v4i ahi[T::TI][2];  // INT8 high codes, one 16-byte operand per matrix instruction
};

template <typename T, bool LO, bool HI>
__device__ __forceinline__ void read_frags(Frags<T>& f, const char* stage, int g, int wm, int wn, int lane) {
  const int r = lane & 31, h = lane >> 5;
#pragma unroll
  for (int j = 0; j < T::TJ; ++j)
    f.bw[j] = *reinterpret_cast<const v4u*>(stage + T::B_OFF + off4(wn * T::WN + j * 32 + r, 2 * g + h));
#pragma unroll
  for (int i = 0; i < T::TI; ++i) {
    const int row = wm * T::WM + i * 32 + r;
    if (LO) f.alo[i] = *reinterpret_cast<const v4u*>(stage + T::A_LO + off4(row, 2 * g + h));
    if (HI) {
      f.ahi[i][0] = *reinterpret_cast<const v4i*>(stage + T::A_HI + off8(row, 4 * g + 2 * h));
      f.ahi[i][1] = *reinterpret_cast<const v4i*>(stage + T::A_HI + off8(row, 4 * g + 2 * h + 1));
    }
  }
}

// Widened operands of one 32-channel slice of the fragments.
template <typename T>
struct Wide {
  v4i bw[T::TJ];
  v4i alo[T::TI];
};

template <typename T, bool LO>
__device__ __forceinline__ void widen_slice(Wide<T>& w, const Frags<T>& f, int s) {
#pragma unroll
  for (int j = 0; j < T::TJ; ++j) w.bw[j] = widen(f.bw[j], s);
  if (LO) {
#pragma unroll
    for (int i = 0; i < T::TI; ++i) w.alo[i] = widen(f.alo[i], s);
  }
}

// The matrix instructions of one 32-channel slice (s = 0/1): 2 * TI * TJ of them, all independent.  The weights are the
// row operand: a lane then holds the outputs of one token, four consecutive channels at a time.
template <typename T, bool LO, bool HI>
__device__ __forceinline__ void mma_slice(const Wide<T>& w, const Frags<T>& f, int s, v16i (&acc_lo)[T::TI][T::TJ],
                                          v16i (&acc_hi)[T::TI][T::TJ]) {
#pragma unroll
  for (int i = 0; i < T::TI; ++i) {
#pragma unroll
    for (int j = 0; j < T::TJ; ++j) {
      if (LO) acc_lo[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w.bw[j], w.alo[i], acc_lo[i][j], 0, 0, 0);
      if (HI) acc_hi[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w.bw[j], f.ahi[i][s], acc_hi[i][j], 0, 0, 0);
    }
  }
}

// Scheduling recipe for one slice: every matrix instruction is followed by a few of the other
// instructions of the region (a wave issues in order, so whatever is not tucked behind a matrix
// instruction leaves the matrix pipeline idle).  VMEM / DS: how many of the first slots also take
// one LDS-direct load / one LDS read.
template <int NMFMA, int VALU, int SALU, int VMEM, int DS>
__device__ __forceinline__ void interleave() {
#pragma unroll
  for (int k = 0; k < NMFMA; ++k) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if (VALU) __builtin_amdgcn_sched_group_barrier(0x002, VALU, 0);
    if (SALU) __builtin_amdgcn_sched_group_barrier(0x004, SALU, 0);
    if (k < VMEM) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    if (k < DS) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
}

// One iteration of the K loop (see k_loop): four slices of 32 channels.  While the matrix
// instructions of a slice run, the operands of the following slice are widened, and the packed
// operands of the slice after that are fetched from LDS, so nothing a matrix instruction needs was
// requested less than a slice (about 500 cycles) earlier.
//   on entry: f0 = fragments of (step kt, channels 0-63), w0 = its slice 0, widened
//   slice A: multiply w0     | fetch f1 = (step kt, channels 64-127), widen f0 slice 1 -> w1
//   slice B: multiply w1     | enqueue the copy of step kt+2, widen f1 slice 0 -> w0
//   barrier (step kt+1 is complete in LDS, step kt's stage may be overwritten)
//   slice C: multiply w0     | fetch f0 = (step kt+1, channels 0-63), widen f1 slice 1 -> w1
//   slice D: multiply w1     | widen f0 slice 0 -> w0
// FILL: 0 = nothing to copy, 1 = the copy of step kt + NS - 1 is enqueued, 2 = the same and that step may be
// partial; ALLOW: K steps whose copies may still be in flight at the barrier (those after step kt+1);
// NEXT: step kt+1 exists.
template <typename T, bool LO, bool HI, int FILL, int ALLOW, bool NEXT>
__device__ __forceinline__ void k_iteration(const Pipe<T, LO, HI>& pipe, char* lds, int kt, int st_cur, int wm, int wn,
                                            int lane, Frags<T>& f0, Frags<T>& f1, Wide<T>& w0, Wide<T>& w1,
                                            v16i (&acc_lo)[T::TI][T::TJ], v16i (&acc_hi)[T::TI][T::TJ]) {
  constexpr int NL = Pipe<T, LO, HI>::NLOAD;
  constexpr int NM = (LO ? 1 : 0) * T::TI * T::TJ + (HI ? 1 : 0) * T::TI * T::TJ;  // matrix instructions per slice
  constexpr int NR = T::TJ + (LO ? T::TI : 0) + (HI ? 2 * T::TI : 0);               // LDS reads per fragment set
  const int st_next = st_cur == T::NS - 1 ? 0 : st_cur + 1;
  const int st_fill = st_cur == 0 ? T::NS - 1 : st_cur - 1;  // the stage of step kt - 1, read for the last time before the previous barrier
  // slice A
  read_frags<T, LO, HI>(f1, lds + st_cur * T::STAGE, 1, wm, wn, lane);
  widen_slice<T, LO>(w1, f0, 1);
  mma_slice<T, LO, HI>(w0, f0, 0, acc_lo, acc_hi);
  interleave<NM, 4, 0, 0, NR>();
  __builtin_amdgcn_sched_barrier(0);
  // slice B
  if (FILL == 1) pipe.template issue<false>(lds + st_fill * T::STAGE, kt + T::NS - 1);
  if (FILL == 2) pipe.template issue<true>(lds + st_fill * T::STAGE, kt + T::NS - 1);
  widen_slice<T, LO>(w0, f1, 0);
  mma_slice<T, LO, HI>(w1, f0, 1, acc_lo, acc_hi);
  interleave<NM, 6, 3, FILL ? NL : 0, 0>();
  __builtin_amdgcn_sched_barrier(0);
  pipeline_barrier<ALLOW * NL>();
  // slice C
  if (NEXT) read_frags<T, LO, HI>(f0, lds + st_next * T::STAGE, 0, wm, wn, lane);
  widen_slice<T, LO>(w1, f1, 1);
  mma_slice<T, LO, HI>(w0, f1, 0, acc_lo, acc_hi);
  interleave<NM, 4, 0, 0, NEXT ? NR : 0>();
  __builtin_amdgcn_sched_barrier(0);
  // slice D
  if (NEXT) widen_slice<T, LO>(w0, f0, 0);
  mma_slice<T, LO, HI>(w1, f1, 1, acc_lo, acc_hi);
  interleave<NM, 3, 0, 0, 0>();
  __builtin_amdgcn_sched_barrier(0);
}

// K loop over NS LDS stages: the copy of step kt + NS - 1 is enqueued while step kt is multiplied; every wave
// waits for its own copy of step kt+1 in the middle of iteration kt (younger copies stay in flight), the
// workgroup meets at a barrier, and the matrix pipeline has operands in registers on both sides of it (see
// k_iteration).  The last NS iterations are peeled so that the steady-state body has no branches.
// Safety: the stage overwritten by the copy of step kt + NS - 1 held step kt-1, last read before the
// barrier of iteration kt-1, and every wave drains its LDS reads (lgkmcnt 0) before that barrier.
// k_loop_start enqueues the first NS - 1 steps; k_loop expects them enqueued (whatever independent work the
// caller has goes between the two calls, under the latency of those first copies).
template <typename T, bool LO, bool HI>
__device__ __forceinline__ void k_loop_start(const Pipe<T, LO, HI>& pipe, char* lds, int st0 = 0) {
  pipe.template issue<true>(lds + st0 * T::STAGE, 0);
#pragma unroll
  for (int s0 = 1; s0 < T::NS - 1; ++s0)
    if (pipe.steps > s0) pipe.template issue<true>(lds + ((st0 + s0) % T::NS) * T::STAGE, s0);
}

// The last iterations of a K loop, peeled: with R steps left after the current one, the iteration that still
// enqueues a copy (R == NS - 1: the last step, which may be partial), then the ones that only drain.
template <typename T, bool LO, bool HI, int R>
__device__ __forceinline__ void k_loop_tail(const Pipe<T, LO, HI>& pipe, char* lds, int steps, int& kt, int& st, int wm, int wn,
                                            int lane, Frags<T>& f0, Frags<T>& f1, Wide<T>& w0, Wide<T>& w1,
                                            v16i (&acc_lo)[T::TI][T::TJ], v16i (&acc_hi)[T::TI][T::TJ]) {
  constexpr int D = T::NS - 1;
  if (steps - 1 - kt == R) {
    constexpr int FILL = R == D ? 2 : 0;
    constexpr int ALLOW = R == D ? D - 1 : (R > 0 ? R - 1 : 0);
    k_iteration<T, LO, HI, FILL, ALLOW, (R > 0)>(pipe, lds, kt, st, wm, wn, lane, f0, f1, w0, w1, acc_lo, acc_hi);
    st = st == T::NS - 1 ? 0 : st + 1;
    ++kt;
  }
  if constexpr (R > 0) k_loop_tail<T, LO, HI, R - 1>(pipe, lds, steps, kt, st, wm, wn, lane, f0, f1, w0, w1, acc_lo, acc_hi);
}

template <int N, int NL>
__device__ __forceinline__ void first_barrier(int in_flight) {  // in_flight steps enqueued, step 0 must have landed
  if constexpr (N > 1) {
    if (in_flight >= N) {
      pipeline_barrier<(N - 1) * NL>();
      return;
    }
    first_barrier<N - 1, NL>(in_flight);
  } else {
    pipeline_barrier<0>();
  }
}

template <typename T, bool LO, bool HI>
__device__ __forceinline__ void k_loop(const Pipe<T, LO, HI>& pipe, char* lds, int wm, int wn, int lane,
                                       v16i (&acc_lo)[T::TI][T::TJ], v16i (&acc_hi)[T::TI][T::TJ], int st0 = 0) {
  constexpr int NL = Pipe<T, LO, HI>::NLOAD;
  constexpr int D = T::NS - 1;
  const int steps = pipe.steps;
  first_barrier<D, NL>(steps < D ? steps : D);
  Frags<T> f0, f1;
  Wide<T> w0, w1;
  read_frags<T, LO, HI>(f0, lds + st0 * T::STAGE, 0, wm, wn, lane);
  widen_slice<T, LO>(w0, f0, 0);
  int st = st0, kt = 0;
  for (; kt + D + 1 < steps; ++kt) {  // steady state: copies of full steps only, D - 1 steps in flight at the barrier
    k_iteration<T, LO, HI, 1, D - 1, true>(pipe, lds, kt, st, wm, wn, lane, f0, f1, w0, w1, acc_lo, acc_hi);
    st = st == T::NS - 1 ? 0 : st + 1;
  }
  k_loop_tail<T, LO, HI, D>(pipe, lds, steps, kt, st, wm, wn, lane, f0, f1, w0, w1, acc_lo, acc_hi);
  __syncthreads();  // the stages are reused by the next loop / the epilogue
}

// Orders this wave's LDS writes before its later LDS reads of other lanes' data (compiler barrier +
// wait for the wave's outstanding LDS operations); no other wave is involved.
__device__ __forceinline__ void wave_lds_fence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((15) | (7 << 4) | (0 << 8) | (3 << 14));  // lgkmcnt(0)
  asm volatile("" ::: "memory");
}

// Epilogue: Y = (acc_lo * s_lo[m] + acc_hi * s_hi[m]) * s_w[n], in this order, in fp32.
// Accumulator register r of lane l of a 32x32 tile is channel 8*(r/4) + 4*(l/32) + r%4 of token l%32.  The finished
// outputs go through LDS (free after the K loops), four channels at a time: every wave transposes 32 tokens x WN channels
// and then stores 16 bytes per lane, whole row segments at once.  (With the tokens as rows a lane held single elements
// of many rows and wrote them to LDS 2 bytes at a time: [4096,4096] x [22016,4096] 552 -> 540 us, the single-product
// kernel 282 -> 264 us.)
// The scales a thread contributes to the epilogue, fetched at the start of the kernel so that their
// latency hides under the K loop.
template <typename T>
struct EpiScales {
  float slo[T::TI], shi[T::TI];  // s_lo and s_hi of this lane's token in each of the wave's 32-token tiles
  float sw;                      // thread t < BN: s_w of channel n0 + t
};

template <typename T>
__device__ __forceinline__ void load_epi_scales(EpiScales<T>& e, const GemmArgs& g, int m0, int n0, int wm, int lane) {
  const int tid = threadIdx.x & (T::NT - 1);
#pragma unroll
  for (int i = 0; i < T::TI; ++i) {
    const int m = min(m0 + wm * T::WM + i * 32 + (lane & 31), g.M - 1);
    e.slo[i] = g.s_lo ? g.s_lo[m] : 0.0f;
    e.shi[i] = g.s_hi[m];
  }
  e.sw = g.s_w[min(n0 + (tid < T::BN ? tid : 0), g.N - 1)];
}

template <typename T, typename OutT>
__device__ __forceinline__ void epilogue_typed(const GemmArgs& g, const EpiScales<T>& es, char* lds,
                                               v16i (&acc_lo)[T::TI][T::TJ], v16i (&acc_hi)[T::TI][T::TJ], int m0, int n0,
                                               int wm, int wn, int wave, int lane) {
  constexpr int ESZ = sizeof(OutT);
  constexpr int ROW = T::WN * ESZ + 16;   // padded row of the transposition buffer (bytes)
  constexpr int PER16 = 16 / ESZ;         // outputs per 16-byte store
  constexpr int CHUNKS = T::WN / PER16;   // 16-byte chunks per row
  constexpr int ROWS_PER_PASS = 64 / CHUNKS;
  constexpr int SC_BYTES = T::BN * 4;     // s_w
  static_assert(T::BN <= T::NT, "one scale per thread");
  static_assert(SC_BYTES + T::NT / 64 * 32 * ROW <= T::LDS_BYTES, "transposition buffers must fit in the stage memory");
  const int tid = threadIdx.x & (T::NT - 1);
  float* sc = reinterpret_cast<float*>(lds);
  char* tb = lds + SC_BYTES + wave * (32 * ROW);
  if (tid < T::BN) sc[tid] = es.sw;
  // workgroup barrier without the memory fence of __syncthreads(): only LDS traffic has to be ordered here
  pipeline_barrier<63>();
  const bool vec_ok = (g.ldy % PER16) == 0;  // rows of Y stay 16-byte aligned
  OutT* yout = reinterpret_cast<OutT*>(g.y);
#pragma unroll
  for (int i = 0; i < T::TI; ++i) {
#pragma unroll
    for (int j = 0; j < T::TJ; ++j) {
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        const int c0 = j * 32 + 8 * rq + 4 * (lane >> 5);  // 4 consecutive channels of the wave's: registers 4 rq + e
        // (clang vector types, not HIP's float4: the compiler orders reads of the latter after every LDS-direct
        // load in flight with a full vmcnt(0) wait)
        const f32x4 sw = *reinterpret_cast<const f32x4*>(sc + wn * T::WN + c0);
        f32x4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          // the accumulators carry the widening factors 256 and 16: shifted out exactly, as integers
          float t = __fmul_rn(static_cast<float>(acc_lo[i][j][4 * rq + e] >> 8), es.slo[i]);
          t = __fmaf_rn(static_cast<float>(acc_hi[i][j][4 * rq + e] >> 4), es.shi[i], t);
          y[e] = __fmul_rn(t, sw[e]);
        }
        char* dst = tb + (lane & 31) * ROW + c0 * ESZ;
        if constexpr (ESZ == 2)
          *reinterpret_cast<v2u*>(dst) = v2u{bf16_rne(y[0]) | static_cast<unsigned>(bf16_rne(y[1])) << 16,
                                             bf16_rne(y[2]) | static_cast<unsigned>(bf16_rne(y[3])) << 16};
        else
          *reinterpret_cast<f32x4*>(dst) = y;
      }
    }
    wave_lds_fence();  // the buffer is private to the wave: its LDS operations execute in order
#pragma unroll
    for (int pass = 0; pass < 32 / ROWS_PER_PASS; ++pass) {
      const int rl = pass * ROWS_PER_PASS + lane / CHUNKS, ch = lane % CHUNKS;
      const int m = m0 + wm * T::WM + i * 32 + rl;
      const int n = n0 + wn * T::WN + ch * PER16;
      if (m < g.M && n < g.N) {
        OutT* dst = yout + static_cast<int64_t>(m) * g.ldy + n;
        if (vec_ok && n + PER16 <= g.N) {
          // streaming store (nt): Y is written once and not read by this kernel; measured 2 % on the
          // single-product kernel, neutral on the two-product one.  Written as asm, so the two idle slots a
          // wide store needs before its data registers may be overwritten are added by hand.
          const v4u vv = *reinterpret_cast<const v4u*>(tb + rl * ROW + ch * 16);
          asm volatile("global_store_dwordx4 %0, %1, off nt\n\ts_nop 1" ::"v"(dst), "v"(vv) : "memory");
        } else {  // ragged right edge or unaligned rows: element by element, straight from LDS
          const OutT* src = reinterpret_cast<const OutT*>(tb + rl * ROW + ch * 16);
          for (int q = 0; q < PER16 && n + q < g.N; ++q) dst[q] = src[q];
        }
      }
    }
    wave_lds_fence();
  }
  if (g.acc_lo_dbg || g.acc_hi_dbg) {  // test hook: the exact accumulators, written element by element
#pragma unroll
    for (int i = 0; i < T::TI; ++i)
#pragma unroll
      for (int j = 0; j < T::TJ; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = m0 + wm * T::WM + i * 32 + (lane & 31);
          const int n = n0 + wn * T::WN + j * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          if (m < g.M && n < g.N) {
            if (g.acc_lo_dbg) g.acc_lo_dbg[static_cast<int64_t>(m) * g.N + n] = acc_lo[i][j][r] >> 8;
            if (g.acc_hi_dbg) g.acc_hi_dbg[static_cast<int64_t>(m) * g.N + n] = acc_hi[i][j][r] >> 4;
          }
        }
  }
}

template <typename T>
__device__ __forceinline__ void epilogue(const GemmArgs& g, const EpiScales<T>& es, char* lds,
                                         v16i (&acc_lo)[T::TI][T::TJ], v16i (&acc_hi)[T::TI][T::TJ], int m0, int n0, int wm,
                                         int wn, int wave, int lane) {
  if (g.out_bf16) epilogue_typed<T, uint16_t>(g, es, lds, acc_lo, acc_hi, m0, n0, wm, wn, wave, lane);
  else epilogue_typed<T, float>(g, es, lds, acc_lo, acc_hi, m0, n0, wm, wn, wave, lane);
}

// Adds the K groups' partial sums (integers: exact in any order) into the first group's registers, through LDS.
// Every stage has been read for the last time (k_loop ends with a barrier); on return LDS is free again.
template <typename T, bool LO>
__device__ __forceinline__ void join_groups(char* lds, int grp, int wave, int lane, v16i (&acc_lo)[T::TI][T::TJ],
                                            v16i (&acc_hi)[T::TI][T::TJ]) {
  constexpr int PER_WAVE = T::TI * T::TJ * 8 * 1024;  // two products, 16 registers of 64 lanes
  auto at = [&](int g, int i, int j, int p, int q) {
    return reinterpret_cast<v4i*>(lds + ((g - 1) * (T::NT / 64) + wave) * PER_WAVE + (((i * T::TJ + j) * 2 + p) * 4 + q) * 1024 + lane * 16);
  };
  if (grp != 0) {
#pragma unroll
    for (int i = 0; i < T::TI; ++i)
#pragma unroll
      for (int j = 0; j < T::TJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (LO) *at(grp, i, j, 0, q) = v4i{acc_lo[i][j][4 * q], acc_lo[i][j][4 * q + 1], acc_lo[i][j][4 * q + 2], acc_lo[i][j][4 * q + 3]};
          *at(grp, i, j, 1, q) = v4i{acc_hi[i][j][4 * q], acc_hi[i][j][4 * q + 1], acc_hi[i][j][4 * q + 2], acc_hi[i][j][4 * q + 3]};
        }
  }
  __syncthreads();
  if (grp == 0) {
#pragma unroll
    for (int g = 1; g < T::S; ++g)
#pragma unroll
      for (int i = 0; i < T::TI; ++i)
#pragma unroll
        for (int j = 0; j < T::TJ; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const v4i h = *at(g, i, j, 1, q);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc_hi[i][j][4 * q + e] += h[e];
            if (LO) {
              const v4i l = *at(g, i, j, 0, q);
#pragma unroll
              for (int e = 0; e < 4; ++e) acc_lo[i][j][4 * q + e] += l[e];
            }
          }
  }
  __syncthreads();  // the epilogue reuses the space
}

// MODE 0: dynamic (low + zero-padded high in one K loop); 1: static (low loop over K or K_lo, then the compact high loop
// over K_hi); 2: one INT8 operand (tied scales, plain W4A8).
template <typename T, int MODE>
__global__ __launch_bounds__(T::THREADS) void gemm_kernel(GemmArgs g) {
  extern __shared__ __attribute__((aligned(16))) char lds_all[];
  const int tid = threadIdx.x & (T::NT - 1);
  const int grp = T::S == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / T::NT);
  const int lane = tid & 63, wave = tid >> 6;
  char* lds = lds_all + grp * (T::NS * T::STAGE);  // every K group has its own stages
  const int wm = wave / T::NWN, wn = wave % T::NWN;
  int tm, tn;
  tile_of_block(blockIdx.x, (g.M + T::BM - 1) / T::BM, (g.N + T::BN - 1) / T::BN, tm, tn);
  if (tm < 0) return;
  const int m0 = tm * T::BM, n0 = tn * T::BN;

  // Order: scales first (they are the oldest vector-memory operations, so no later wait is held up by
  // them), then the first copies of the K loop, then the accumulators are cleared under their latency.
  EpiScales<T> es;
  load_epi_scales<T>(es, g, m0, n0, wm, lane);
  constexpr bool HI1 = MODE == 0;  // the first loop also carries the INT8 operand (dynamic mode)
  Pipe<T, true, HI1> p1;           // MODE 0: low + zero-padded high; MODE 1: low only; MODE 2: unused
  Pipe<T, false, true> p2;         // MODE 1, 2: the compact high loop
  if constexpr (MODE == 0) {
    p1.init(g.a_lo, g.K / 2, g.a_hi_dense, g.K, g.wq, g.K / 2, g.K, m0, n0, g.M, g.N, blockIdx.x & 7);
    k_loop_start<T, true, HI1>(p1, lds);
  } else if constexpr (MODE == 1) {
    p1.init(g.a_lo, g.K_lo / 2, nullptr, 0, g.w_lo, g.K_lo / 2, g.K_lo, m0, n0, g.M, g.N, blockIdx.x & 7);
    k_loop_start<T, true, HI1>(p1, lds);
  } else {
    p2.init(nullptr, 0, g.a_hi_compact, g.lda_hi_compact, g.w_hi, g.K_hi / 2, g.K_hi, m0, n0, g.M, g.N, blockIdx.x & 7);
    k_loop_start<T, false, true>(p2, lds);
  }

  v16i acc_lo[T::TI][T::TJ], acc_hi[T::TI][T::TJ];
#pragma unroll
  for (int i = 0; i < T::TI; ++i)
#pragma unroll
    for (int j = 0; j < T::TJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc_lo[i][j][r] = 0;
        acc_hi[i][j][r] = 0;
      }

  if constexpr (MODE == 0) {
    k_loop<T, true, HI1>(p1, lds, wm, wn, lane, acc_lo, acc_hi);
  } else {
    if constexpr (MODE == 1) {
      k_loop<T, true, HI1>(p1, lds, wm, wn, lane, acc_lo, acc_hi);
      p2.init(nullptr, 0, g.a_hi_compact, g.lda_hi_compact, g.w_hi, g.K_hi / 2, g.K_hi, m0, n0, g.M, g.N, blockIdx.x & 7);
      k_loop_start<T, false, true>(p2, lds);
    }
    k_loop<T, false, true>(p2, lds, wm, wn, lane, acc_lo, acc_hi);
  }

  if constexpr (T::S > 1) {
    join_groups<T, MODE != 2>(lds_all, grp, wave, lane, acc_lo, acc_hi);
    if (grp != 0) {
      pipeline_barrier<63>();  // the epilogue's
      return;
    }
  }
  epilogue<T>(g, es, lds, acc_lo, acc_hi, m0, n0, wm, wn, wave, lane);
}

template <typename T, int MODE>
int launch_mode(const GemmArgs& g, hipStream_t st) {
  const int tiles = ((g.N + T::BN - 1) / T::BN) * ((g.M + T::BM - 1) / T::BM);
  const int blocks = (tiles + 7) / 8 * 8;
  hipLaunchKernelGGL((gemm_kernel<T, MODE>), dim3(blocks), dim3(T::THREADS), T::LDS_BYTES, st, g);
  return hipGetLastError() == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}


// Three stages everywhere: a fourth stage for the 128x256 tile (exactly the 160 KB of LDS) was timed and changes
// nothing (c3: 680 us either way on dense random operands) -- the copies are not what the loop waits for.
typedef Tile<128, 256, 2, 4> Big;                  // matrix-core bound shapes
typedef Tile<128, 128, 4, 2> Mid;                  // too few of those to occupy every compute unit
typedef Tile<64, 128, 2, 2, true, 2> SmallWide;  // fewer still: two K groups of four waves per workgroup, so that a compute
typedef Tile<64, 64, 2, 2, true, 2> Small;       // unit has two waves per SIMD although it has one workgroup
typedef Tile<64, 64, 2, 2> Light;                // short K: one K group of four waves, three workgroups per compute unit
typedef Tile<256, 256, 2, 4, false> Huge;  // single-product modes on large shapes: with one accumulator set a wave
                                           // holds 128 x 64 outputs, which halves the operand traffic and the
                                           // widening arithmetic per matrix instruction

enum Variant { V_HUGE, V_BIG, V_MID, V_SMALL_WIDE, V_SMALL, V_FEW, V_LIGHT };

// Measured times in us, up to 4096 channels, k = channels / 1024; [mode] as in GemmArgs' kernels: two products, static, one
// product.  A tile that fills a compute unit: launch + rounds * (round + per_k * k).  The light tile: the same with a term for
// every tile of a compute unit and one for every three.  The few-token kernel: the same with a term for its rows times its
// channel tiles, over 32 rows.  (Fitted to about 1450 shapes of 1 to 4096 tokens and 64 to 4096 channels, within 10 %.)
struct TileTime { float launch, round, per_k; };
struct SharedTime { float launch, each, each_k, group, group_k; };
constexpr TileTime kBigTime[3] = {{0.16f, 6.29f, 8.00f}, {0.71f, 6.67f, 5.15f}, {0.25f, 5.21f, 4.47f}};
constexpr TileTime kMidTime[3] = {{1.10f, 4.07f, 5.03f}, {1.45f, 4.57f, 3.47f}, {1.13f, 3.26f, 3.51f}};
constexpr TileTime kSmallWideTime[3] = {{1.51f, 4.23f, 2.88f}, {1.84f, 4.89f, 2.02f}, {1.53f, 3.49f, 1.99f}};
constexpr TileTime kSmallTime[3] = {{1.67f, 2.49f, 1.92f}, {1.73f, 3.24f, 1.26f}, {1.70f, 2.17f, 1.36f}};
constexpr SharedTime kLightTime[3] = {{2.51f, 0.49f, 1.36f, 0.61f, 1.09f}, {3.01f, 0.68f, 0.67f, 0.47f, 1.42f}, {2.29f, 0.29f, 0.88f, 0.93f, 0.98f}};
constexpr SharedTime kFewTime[3] = {{1.94f, 0.37f, 0.36f, 1.25f, 0.34f}, {2.23f, 0.46f, 0.29f, 1.00f, 0.31f}, {1.94f, 0.32f, 0.26f, 1.07f, 0.31f}};

// Which kernel a shape runs on.  Every tile kernel but the light one fills a compute unit with one workgroup, so a launch takes
// ceil(tiles / 256) rounds, and a round of each tile its own time: at K = 4096, two products, 46 us (Big), 27 us
// (Mid), 18 us (SmallWide), 11.5 us (Small); single product 32 / 18.5 / 13.5 / 9 us.  The least rounds x time wins, a
// larger tile on near ties (it moves less data).  Measured against the old rule (Big above 128 of its tiles, else Mid;
// 64x64 up to 64 tokens): [333,11008] x [4095,11008] 66.9 -> 42.2 us (SmallWide), [128,4096] x [12288,4096] 26.7 ->
// 18.2 us, [64,8192] x [28672,8192] 47.5 -> 36.0 us (SmallWide), [512,4096] x [4096,4096] 27.2 -> 19.7 us.
// With short K a workgroup's start and epilogue count for more than its K steps, and only several workgroups on a compute unit
// hide them: up to 4096 channels and 1024 tiles the light tile is taken where the times above say that it is 5 % ahead (with
// more tiles its narrow rows of Y cost more than it gains where they are unaligned or fp32: [2523,128] x [4649,128] 33.8 us
// against 29.4 us with Mid).  [64,512] x [20000,512] 7.4 us (SmallWide) -> 5.8 us, [32,64] x [28672,64] 6.8 us (few tokens) -> 4.4 us, [512,1024] x [4096,1024] 9.8 ->
// 8.2 us; but [64,4096] x [12288,4096] 11.7 us (Small) against 14.5 us.
Variant pick_variant(int M, int N, int K, int mode) {
  const bool single = mode == 2;
  auto tiles = [&](int bm, int bn) { return static_cast<int64_t>((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  if (single && tiles(256, 256) >= kHugeMinTiles) return V_HUGE;
  const float k = K / 1024.0f;
  const int64_t each = (tiles(64, 64) + 255) / 256;
  auto shared = [&](const SharedTime& t, float n, float groups) {
    return t.launch + n * (t.each + t.each_k * k) + groups * (t.group + t.group_k * k);
  };
  const float light = K > 4096 || each > 4 ? 1e30f : shared(kLightTime[mode], each, (each + 2) / 3);
  if (gemm_few_supports(M, N)) {
    int rows, ct;
    gemm_few_shape(M, N, &rows, &ct);
    const float rounds = ((N + 16 * ct - 1) / (16 * ct) + 255) / 256;
    return light < 0.95f * shared(kFewTime[mode], rounds * rows * ct / 32.0f, rounds) ? V_LIGHT : V_FEW;
  }
  struct { Variant v; int bm, bn, two, one; const TileTime* t; } const t[] = {{V_BIG, 128, 256, 460, 320, kBigTime},
                                                                              {V_MID, 128, 128, 270, 185, kMidTime},
                                                                              {V_SMALL_WIDE, 64, 128, 180, 135, kSmallWideTime},
                                                                              {V_SMALL, 64, 64, 115, 90, kSmallTime}};
  Variant best = V_BIG;
  int64_t least = INT64_MAX;
  float time = 0.0f;
  for (const auto& c : t) {
    const int64_t rounds = (tiles(c.bm, c.bn) + 255) / 256, cost = rounds * (single ? c.one : c.two);
    if (least == INT64_MAX || cost * 10 < least * 9) {
      least = cost;
      best = c.v;
      time = c.t[mode].launch + rounds * (c.t[mode].round + c.t[mode].per_k * k);
    }
  }
  return light < 0.95f * time ? V_LIGHT : best;
}

template <typename T, int MODE>
hipError_t raise_lds_limit() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_kernel<T, MODE>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
}

template <int MODE>
int launch_for_mode(const GemmArgs& g, hipStream_t st, Variant v) {
  switch (v) {
    case V_FEW: return launch_gemm_few(g, MODE, st);
    case V_HUGE:
      if constexpr (MODE == 2) return launch_mode<Huge, 2>(g, st);
      return SQ_ERR_UNSUPPORTED;  // pick_variant gives it to single-product calls only
    case V_BIG: return launch_mode<Big, MODE>(g, st);
    case V_MID: return launch_mode<Mid, MODE>(g, st);
    case V_SMALL_WIDE: return launch_mode<SmallWide, MODE>(g, st);
    case V_LIGHT: return launch_mode<Light, MODE>(g, st);
    default: return launch_mode<Small, MODE>(g, st);
  }
}

}  // namespace

// The GEMM kernels use more dynamic LDS than the default limit; the limit of every instantiation is raised
// here, once per device (called by the library's per-device initialisation, never on the launch path).
int init_gemm_kernels() {
  hipError_t e = hipSuccess;
#define SQ_RAISE(T)                                          \
  if (e == hipSuccess) e = raise_lds_limit<T, 0>();          \
  if (e == hipSuccess) e = raise_lds_limit<T, 1>();          \
  if (e == hipSuccess) e = raise_lds_limit<T, 2>();
  SQ_RAISE(Big) SQ_RAISE(Mid) SQ_RAISE(SmallWide) SQ_RAISE(Small) SQ_RAISE(Light)
#undef SQ_RAISE
  if (e == hipSuccess) e = raise_lds_limit<Huge, 2>();
  return e == hipSuccess ? init_gemm_few_kernels() : SQ_ERR_LAUNCH;
}

// What sq_gemm_variant reports: the choice launch_gemm makes.
const char* gemm_variant_name(int M, int N, int K, int mode) {
  switch (pick_variant(M, N, K, mode)) {
    case V_HUGE: return "tile256x256";
    case V_BIG: return "tile128x256";
    case V_MID: return "tile128x128";
    case V_SMALL_WIDE: return "tile64x128";
    case V_SMALL: return "tile64x64";
    case V_LIGHT: return "tile64x64_light";
    default: return "few_tokens";
  }
}

int launch_gemm(const GemmArgs& g, hipStream_t st) {
  if (g.a_lo && g.a_hi_dense) return launch_for_mode<0>(g, st, pick_variant(g.M, g.N, g.K, 0));
  if (g.a_lo && g.a_hi_compact) return launch_for_mode<1>(g, st, pick_variant(g.M, g.N, g.K, 1));
  if (!g.a_lo && g.a_hi_compact) return launch_for_mode<2>(g, st, pick_variant(g.M, g.N, g.K, 2));
  return SQ_ERR_UNSUPPORTED;
}

}  // namespace sq
