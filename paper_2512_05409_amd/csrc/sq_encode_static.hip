// sq_encode, static rule (Algorithm 2: the high-precision channels of every bank are fixed for all tokens by
// a calibrated channel mask), row-staged kernel for gfx950.
//
// With a static mask the selection costs nothing and the work is a gather: the paper's GPU path (Section 3.3)
// reorders the weights by the mask ahead of time so that at run time "only selection and gathering" is left on
// the activation side.  This kernel therefore writes, besides the format's own arrays, the activations in that
// reordered form: `lo_compact`, the low codes of the low channels only (K_lo = K - K_hi of them, ascending
// channel order), next to `hi_val`, the high codes of the high channels only -- the two operands of the two
// products, each contiguous, so that the low product runs over K_lo channels instead of K.
//
// A workgroup walks over token rows, which LDS-direct loads copy into two row buffers, one row ahead.  A thread owns the
// same 16-byte pieces (8 channels) of every row, so everything that depends on the mask only is worked out once and
// stays in registers: which of the 8 channels are low, the byte permutation that moves their codes together, where in the
// compact row they go, and the LDS offsets of the high channels' values.  Per row a thread reads its pieces (taking the
// row maxima on the way) and, once the workgroup's maxima are combined, quantises them to 8 bytes, moves the low ones
// together (v_perm_b32), packs them to nibbles and ORs them into the compact row in LDS, which leaves in 16-byte stores.
// Bounds: HBM (2 bytes read and 0.5 (1 - k/b) + k/b written per element) and vector arithmetic (about 7 instructions
// per element) are close to each other: another row costs 5.9 ns at 11008 channels (4.8 TB/s), launch, tables and the
// first row about 10 us.  Gathering every low code by its own 16-bit LDS read instead was bound by those reads and their
// bank conflicts, and building the index table one bank per thread took most of a short call: [4096,11008] 43.6 -> 34.6
// us, [4096,4096] 40.2 -> 17.4 us, [2048,14336] 41.4 -> 24.2 us, [8,11008] 15.3 -> 9.2 us (calls back to back).
#include "sq_encode_common.h"

namespace sq {
namespace {

using namespace enc;

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// max of two pairs of 16-bit magnitudes, both halves in one instruction (v_pk_max_u16)
__device__ __forceinline__ uint32_t pk_max_u16(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}

struct GatherArgs {
  const uint16_t* x;
  int64_t ldx;
  int M, K, B, kt;
  int K_hi, K_lo;
  int bufs;               // row buffers: 2, or 1 where two do not fit
  const uint32_t* mask;   // [K/32]
  uint8_t* d_lo;          // [M, K/2] dense low codes, or null
  uint8_t* lo_compact;    // [M, K_lo/2], or null
  int8_t* hi_val;         // [M, K_hi]
  float* s_lo;
  float* s_hi;
  float q_hi, q_lo;       // largest code magnitudes of the two parts (127 and 7 for the 8/4 pair)
};

// At most n vector-memory operations outstanding.  n is known at run time only (and the same for the whole wave);
// the instruction takes a constant, so n is rounded down to one of a few.
template <int N>
__device__ __forceinline__ void wait_vm_at_most(int n) {
  if constexpr (N > 0) {
    if (n < N) {
      wait_vm_at_most<N - (N > 8 ? 4 : 1)>(n);
      return;
    }
  }
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
// Workgroup barrier that orders LDS traffic only (__syncthreads() would also drain the copies in flight).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((15) | (7 << 4) | (0 << 8) | (3 << 14));  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ uint32_t lds_u16(const char* lds, uint32_t addr) {
  return *reinterpret_cast<const uint16_t*>(lds + addr);
}

// *p |= v.  (Written out: before an atomic on LDS the compiler waits for every LDS-direct load in flight.)
__device__ __forceinline__ void lds_or(uint32_t* p, uint32_t v) {
  const uint32_t at = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint32_t*)p));
  asm volatile("ds_or_b32 %0, %1" ::"v"(at), "v"(v) : "memory");
}

// The low bytes of the rounded products of 8 consecutive channels (4 packed bf16 pairs), two dwords.
__device__ __forceinline__ void quant8(const uint32_t* pairs, float inv, uint32_t& b03, uint32_t& b47) {
  b03 = b47 = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint32_t w = pairs[e >> 1];
    const float xf = __uint_as_float((e & 1) ? (w & 0xFFFF0000u) : (w << 16));
    uint32_t& d = e < 4 ? b03 : b47;
    d = __builtin_amdgcn_alignbit(__float_as_uint(__fadd_rn(__fmul_rn(xf, inv), kRoundMagic)), d, 8);
  }
}

// LDS: the row buffers [K * 2], the compact row [K_lo / 2 + 16], the mask [K / 8].
// NT: threads; IT: pieces a thread owns at most (with 3, registers for three workgroups per compute unit, which is what
// LDS holds of such rows: 34.6 us with three, 35.9 us with two at 11008 channels, although 4 of the 80 registers are spilled
// then, and 21 where both forms of the low part are written).  COMPACT / DENSE: lo_compact / d_lo are written.
template <int NT, int IT, bool COMPACT, bool DENSE>
__global__ __launch_bounds__(NT, IT == 3 ? 6 : 1) void encode_static_gather_kernel(GatherArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  constexpr int NWAVE = NT / 64;
  static_assert(NWAVE == 1 || NWAVE % 4 == 0, "the maxima are combined four waves at a time");
  __shared__ __attribute__((aligned(16))) uint32_t part[2][NWAVE];  // row maxima of the waves: high << 16 | low
  const int row_bytes = 2 * a.K;
  uint32_t* out_sh = reinterpret_cast<uint32_t*>(lds + a.bufs * row_bytes);
  uint32_t* mask_sh = out_sh + a.K_lo / 8 + 4;
  uint32_t* lut = mask_sh + a.K / 32;  // [256][2] byte permutation of every mask byte
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  const int chunks = a.K / 8;  // 16-byte pieces of a row
  const int out16 = a.K_lo / 32, n_hi = a.K_hi / 4;  // 16-byte pieces of the compact row, dwords of high codes
  const int it_p = (chunks + NT - 1) / NT, it_hi = (n_hi + NT - 1) / NT;  // uniform
  // instructions of this wave over n items dealt to the threads in turn: those that have a lane with an item
  auto mine = [&](int n) { return (n - wave * 64 + NT - 1) / NT; };
  const int n_copy = mine(chunks), n_store = mine(n_hi) + (COMPACT ? mine(out16) : 0) + (DENSE ? mine(chunks) : 0);

  // thread t copies pieces t, t + NT, ... (1 KB of consecutive memory per wave instruction)
  auto stage_row = [&](int64_t m, int buf) {
    const char* xrow = reinterpret_cast<const char*>(a.x + m * a.ldx);
    char* row = lds + buf * row_bytes;
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int c = i * NT + tid;
      if (c < chunks) __builtin_amdgcn_global_load_lds(xrow + c * 16, (lds_ptr_t)(row + (i * NT + wave * 64) * 16), 16, 0, 0);
    }
  };

  const int64_t stride = gridDim.x;
  if (a.bufs == 2) stage_row(blockIdx.x, 0);  // the grid has at most M workgroups

  // ---- once per workgroup ----
  for (int w = tid; w < a.K / 32; w += NT) mask_sh[w] = a.mask[w];
  for (int w = tid; w < a.K_lo / 8 + 4; w += NT) out_sh[w] = 0;
  uint16_t* tab_hi = reinterpret_cast<uint16_t*>(lds + (a.bufs - 1) * row_bytes);  // channels of the high positions, in the last buffer
  for (int w = tid; w < a.K_hi / 2; w += NT) reinterpret_cast<uint32_t*>(tab_hi)[w] = 0;  // (a malformed mask leaves gaps)
  auto moves = [](uint32_t mask8) {  // moves the bytes whose mask bit is clear together; 0x0C selects a zero byte
    uint64_t s = 0x0C0C0C0C0C0C0C0Cull;
    for (int e = 7; e >= 0; --e)
      if (!((mask8 >> e) & 1)) s = (s << 8) | static_cast<uint64_t>(e);
    return s;
  };
  if (COMPACT && NT >= 256 && tid < 256) {
    const uint64_t s = moves(tid);
    lut[2 * tid] = static_cast<uint32_t>(s);
    lut[2 * tid + 1] = static_cast<uint32_t>(s >> 32);
  }
  lds_barrier();
  const int nlo = a.B - a.kt, lgB = 31 - __clz(a.B);
  // of the thread's pieces: byte permutation, first compact position, mask bits, magnitude bits of the low channels
  uint32_t sel[IT][2], at[IT], mb[IT], keep[IT][4];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    sel[i][0] = sel[i][1] = 0x0C0C0C0Cu;  // a thread past the end of the row ORs zeros
    at[i] = mb[i] = keep[i][0] = keep[i][1] = keep[i][2] = keep[i][3] = 0;
    const int c = i * NT + tid;
    if (c < chunks) {
      const int ch = 8 * c, bank = ch >> lgB, w0 = bank << (lgB - 5), w1 = ch >> 5;
      int hi = 0;  // high channels of the bank before this piece
      for (int w = w0; w < w1; ++w) hi += __popc(mask_sh[w]);
      const uint32_t word = mask_sh[w1];
      hi += __popc(word & ((1u << (ch & 31)) - 1u));
      mb[i] = (word >> (ch & 31)) & 0xFFu;
      // (a malformed mask: positions past the bank's end stay inside the row and its spare dwords)
      at[i] = static_cast<uint32_t>(bank * nlo + min((ch & (a.B - 1)) - hi, nlo));
      if (COMPACT && NT >= 256) {
        sel[i][0] = lut[2 * mb[i]];
        sel[i][1] = lut[2 * mb[i] + 1];
      } else if (COMPACT) {
        const uint64_t s = moves(mb[i]);
        sel[i][0] = static_cast<uint32_t>(s);
        sel[i][1] = static_cast<uint32_t>(s >> 32);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        keep[i][q] = ((mb[i] >> (2 * q)) & 1u ? 0u : 0x7FFFu) | ((mb[i] >> (2 * q + 1)) & 1u ? 0u : 0x7FFF0000u);
      for (uint32_t left = mb[i]; left != 0 && hi < a.kt; left &= left - 1, ++hi)
        tab_hi[bank * a.kt + hi] = static_cast<uint16_t>(ch + __ffs(static_cast<int>(left)) - 1);
    }
  }
  lds_barrier();
  uint32_t ahi[IT][4];  // LDS offsets inside a row buffer
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    if (i < it_hi) {
      const u16x4 v = *reinterpret_cast<const u16x4*>(tab_hi + 4 * min(i * NT + tid, n_hi - 1));
#pragma unroll
      for (int e = 0; e < 4; ++e) ahi[i][e] = 2u * v[e];
    }
  }
  lds_barrier();
  if (a.bufs == 1) stage_row(blockIdx.x, 0);
  else if (blockIdx.x + stride < a.M) stage_row(blockIdx.x + stride, 1);

  int it = 0;
  for (int64_t m = blockIdx.x; m < a.M; m += stride, ++it) {
    // Operations younger than this row's copy: the later rows' copies, and the stores of as many rows as there are buffers
    asm volatile("" ::: "memory");
    wait_vm_at_most<32>((a.bufs == 2 && m + stride < a.M ? n_copy : 0) + min(it, a.bufs) * n_store);
    lds_barrier();  // barrier A: every wave's part of the row is there
    const int buf = a.bufs == 2 ? it & 1 : 0;
    const char* row = lds + buf * row_bytes;

    // ---- the thread's pieces, the high values it owns, and the maxima of their magnitudes (packed: two 15-bit
    // magnitudes per register) ----
    uint32_t v[IT][4], vhi[IT][2];
    uint32_t mx_hi = 0, mx_lo = 0;
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      if (i < it_p) {
        const u32x4 t = *reinterpret_cast<const u32x4*>(row + min(i * NT + tid, chunks - 1) * 16);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[i][q] = t[q];
      }
    }
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      if (i < it_hi) {
#pragma unroll
        for (int q = 0; q < 2; ++q) vhi[i][q] = lds_u16(row, ahi[i][2 * q]) | (lds_u16(row, ahi[i][2 * q + 1]) << 16);
      }
    }
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      if (i < it_p) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          mx_lo = pk_max_u16(mx_lo, v[i][q] & keep[i][q]);
        }
      }
      if (i < it_hi) {
#pragma unroll
        for (int q = 0; q < 2; ++q) mx_hi = pk_max_u16(mx_hi, vhi[i][q] & 0x7FFF7FFFu);
      }
    }
    uint32_t mx = (umax(mx_hi & 0xFFFFu, mx_hi >> 16) << 16) | umax(mx_lo & 0xFFFFu, mx_lo >> 16);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) mx = pk_max_u16(mx, static_cast<uint32_t>(__shfl_xor(static_cast<int>(mx), off, 64)));
    if (NWAVE > 1 && lane == 0) part[it & 1][wave] = mx;
    lds_barrier();  // barrier B: the row has been read for the last time, the waves' maxima are there
    if (m + a.bufs * stride < a.M) stage_row(m + a.bufs * stride, buf);
    if constexpr (NWAVE > 1) {
      mx = 0;
#pragma unroll
      for (int w = 0; w < NWAVE; w += 4) {
        const u32x4 p = *reinterpret_cast<const u32x4*>(&part[it & 1][w]);
        mx = pk_max_u16(pk_max_u16(mx, pk_max_u16(p[0], p[1])), pk_max_u16(p[2], p[3]));
      }
    }
    const uint32_t ah = mx >> 16, al = mx & 0xFFFFu;
    const float amax_hi = __uint_as_float(ah << 16), amax_lo = __uint_as_float(al << 16);
    const float inv_hi = ah ? a.q_hi / amax_hi : 0.0f;
    const float inv_lo = al ? a.q_lo / amax_lo : 0.0f;
    if (tid == 0) {
      a.s_hi[m] = ah ? amax_hi / a.q_hi : 1.0f;
      a.s_lo[m] = al ? amax_lo / a.q_lo : 1.0f;
    }

    // ---- quantise from the registers ----
    uint32_t* dst_hi = reinterpret_cast<uint32_t*>(a.hi_val + m * a.K_hi);
    uint32_t* dst_de = reinterpret_cast<uint32_t*>(a.d_lo + m * (a.K / 2));
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      if (COMPACT && i < it_p) {
        uint32_t b03, b47;
        quant8(v[i], inv_lo, b03, b47);
        uint32_t t0 = __builtin_amdgcn_perm(b47, b03, sel[i][0]) & 0x0F0F0F0Fu;
        uint32_t t1 = __builtin_amdgcn_perm(b47, b03, sel[i][1]) & 0x0F0F0F0Fu;
        t0 |= t0 >> 4;
        t1 |= t1 >> 4;
        const uint64_t x = static_cast<uint64_t>(__builtin_amdgcn_perm(t1, t0, 0x06040200u)) << (4 * (at[i] & 7));
        uint32_t* o = out_sh + (at[i] >> 3);
        lds_or(o, static_cast<uint32_t>(x));
        lds_or(o + 1, static_cast<uint32_t>(x >> 32));
      }
      if (i < it_hi) {
        uint32_t acc = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t w = vhi[i][e >> 1];
          const float xf = __uint_as_float((e & 1) ? (w & 0xFFFF0000u) : (w << 16));
          const float r = __fadd_rn(__fmul_rn(xf, inv_hi), kRoundMagic);
          acc = __builtin_amdgcn_alignbit(__float_as_uint(r), acc, 8);
        }
        if (i * NT + tid < n_hi) dst_hi[i * NT + tid] = acc;
      }
      if (DENSE && i * NT + tid < chunks)
        dst_de[i * NT + tid] = quant_lo8(v[i], inv_lo) & ~spread_bits_to_nibbles(mb[i]);
    }
    if constexpr (COMPACT) {
      lds_barrier();  // barrier C: the compact row is complete
      u32x4* dst = reinterpret_cast<u32x4*>(a.lo_compact + m * (a.K_lo / 2));
#pragma unroll
      for (int i = 0; i < IT; ++i) {
        const int j = i * NT + tid;
        if (j < out16) {
          u32x4* o = reinterpret_cast<u32x4*>(out_sh + 4 * j);
          dst[j] = *o;
          *o = u32x4{0u, 0u, 0u, 0u};  // for the next row, whose codes arrive after two more barriers
        }
      }
    }
  }
}

constexpr size_t kLdsLimit = 158 * 1024;

size_t gather_lds_bytes(const sq_params& p, int bufs) {
  const size_t K_lo = p.K - static_cast<size_t>(p.K / p.bank) * p.topk;
  return static_cast<size_t>(bufs) * 2 * p.K + K_lo / 2 + 16 + p.K / 8 + 2048;
}

// Threads and pieces per thread: rows of up to 512, 1024, 4096, 8192, 12288, 16384 and 40960 channels.  Eight waves: with four
// and twice the pieces [4096,4096] took 24.5 us instead of 17 us (the fixed work per wave and row is spread over less).  But
// waves without channels issue as much as the others: rows of up to 1024 channels are a single wave's ([8192,512] 41.5 -> 7.9 us,
// [8192,64] with b = 32 44 -> 9.5 us, [8,512] 4.8 -> 3.5 us, [8,1024] 4.7 -> 4.4 us).
#define SQ_STATIC_CFG(X) X(64, 1) X(64, 2) X(512, 1) X(512, 2) X(512, 3) X(512, 4) X(512, 10)

template <int NT, int IT>
int launch_it(const GatherArgs& a, int blocks, size_t lds, hipStream_t st) {
  if (!a.d_lo) hipLaunchKernelGGL((encode_static_gather_kernel<NT, IT, true, false>), dim3(blocks), dim3(NT), lds, st, a);
  else if (!a.lo_compact) hipLaunchKernelGGL((encode_static_gather_kernel<NT, IT, false, true>), dim3(blocks), dim3(NT), lds, st, a);
  else hipLaunchKernelGGL((encode_static_gather_kernel<NT, IT, true, true>), dim3(blocks), dim3(NT), lds, st, a);
  return hipGetLastError() == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}

template <int NT, int IT, bool COMPACT, bool DENSE>
hipError_t raise_static() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(encode_static_gather_kernel<NT, IT, COMPACT, DENSE>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLimit);
}

}  // namespace

// Rows of up to about 37000 channels: the bound that callers know, what a row and two tables of 16-bit channel numbers for it
// would take.  (One row buffer and the compact row take a little less.)
bool encode_static_gather_supports(const sq_params& p) {
  if (p.K > 40960) return false;  // pieces per thread; also keeps the channel numbers in 16 bits
  const size_t row = (static_cast<size_t>(p.K) * 2 + 4095) / 4096 * 4096;
  return row + static_cast<size_t>(p.K) * 2 + p.K / 8 + 64 <= 150 * 1024;
}

int init_encode_static_kernels() {
  hipError_t e = hipSuccess;
#define X(NT, IT)                                                      \
  if (e == hipSuccess) e = raise_static<NT, IT, true, false>();        \
  if (e == hipSuccess) e = raise_static<NT, IT, false, true>();        \
  if (e == hipSuccess) e = raise_static<NT, IT, true, true>();
  SQ_STATIC_CFG(X)
#undef X
  return e == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}

int launch_encode_static_gather(const sq_params& p, const uint16_t* x, int64_t ldx, const uint32_t* mask,
                                const sq_act& out, hipStream_t st) {
  GatherArgs a;
  a.x = x;
  a.ldx = ldx;
  a.M = p.M;
  a.K = p.K;
  a.B = p.bank;
  a.kt = p.topk;
  a.K_hi = (p.K / p.bank) * p.topk;
  a.K_lo = p.K - a.K_hi;
  a.mask = mask;
  a.d_lo = out.d_lo;
  a.lo_compact = out.lo_compact;
  a.hi_val = out.hi_val;
  a.s_lo = out.scale_lo;
  a.s_hi = out.scale_hi;
  a.q_hi = code_max(p.h_high, 8);
  a.q_lo = code_max(p.h_low, 4);
  a.bufs = gather_lds_bytes(p, 2) <= kLdsLimit ? 2 : 1;
  const size_t lds = gather_lds_bytes(p, a.bufs);
  // as many workgroups as are resident at once, each walking over its share of the rows
  const int64_t per_cu = static_cast<int64_t>(160 * 1024 / (lds + 64));
  const int64_t most = p.K <= 1024 ? 16 : p.K <= 8192 ? 4 : p.K <= 12288 ? 3 : 2;
  const int64_t cap = device_compute_units() * (per_cu > most ? most : per_cu);
  const int blocks = static_cast<int>(p.M < cap ? p.M : cap);
#define X(NT, IT) \
  if (p.K <= NT * IT * 8) return launch_it<NT, IT>(a, blocks, lds, st);
  SQ_STATIC_CFG(X)
#undef X
  return SQ_ERR_UNSUPPORTED;
}

}  // namespace sq
