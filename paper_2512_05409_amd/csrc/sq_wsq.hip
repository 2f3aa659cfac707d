// SQ-format on WEIGHTS at run time (Section 3.2.1, Algorithm 1, Figure 1's caption; Section 3.3): the W(SQ)A8 /
// W(SQ)A4 linear layer, gfx950.  Every bank of b input channels of every output channel is a quantisation group
// of its own: its k most important weights (I = w^2 / diag(H^-1)^2) are INT8 with one scale, the others INT4 with
// another, and the low part carries the unused code v_mask at the high positions.  The activations are plain
// per-token INT8 (or INT4) codes.
//     Y[m,n] = s_a[m] * sum_g ( acc_lo[m,n,g] * s_lo[n,g] + acc_hi[m,n,g] * s_hi[n,g] )
// The scales change from bank to bank along K, so integer accumulators of different banks cannot be added: each
// bank's two products (exact, on v_mfma_i32_32x32x32_i8) are converted and folded into an fp32 accumulator in a
// fixed order.  That is 5 vector instructions per accumulator register per bank against 4 matrix instructions
// per bank of 64 channels: this layer is bound by vector arithmetic, not by the matrix cores.
#include "sq_gemm_common.h"

namespace sq {
namespace {

using gemm::lds_ptr_t;
using gemm::v2u;
using gemm::v4u;
constexpr float kMagic = 12582912.0f;  // 1.5 * 2^23: adding it leaves rne(x) in the low mantissa bits

__device__ __forceinline__ int rne_code(float x, float inv) {
  // the mantissa field of 1.5 * 2^23 + n is 0x400000 + n
  return static_cast<int>(__float_as_uint(__fadd_rn(__fmul_rn(x, inv), kMagic)) & 0x7FFFFFu) - 0x400000;
}
__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) { return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f)); }

// ---- offline: weights -> SQ-format.  One thread per (output channel, bank) group. ----
template <int B>
__global__ __launch_bounds__(64) void wsq_encode_kernel(const uint16_t* __restrict__ w, int64_t ldw, int N, int K, int kt,
                                                        const float* __restrict__ hinv, float q_hi, float q_lo, int v_mask,
                                                        uint8_t* __restrict__ lo, int8_t* __restrict__ hi_val,
                                                        float* __restrict__ s_lo, float* __restrict__ s_hi) {
  const int G = K / B;
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * 64 + threadIdx.x;
  if (idx >= static_cast<int64_t>(N) * G) return;
  const int64_t n = idx / G;
  const int g = static_cast<int>(idx - n * G);
  const uint16_t* src = w + n * ldw + static_cast<int64_t>(g) * B;
  float wv[B], imp[B];
  for (int i = 0; i < B; ++i) {
    wv[i] = bf16_to_f32(src[i]);
    const float d = hinv ? hinv[g * B + i] : 1.0f;
    imp[i] = __fdiv_rn(__fmul_rn(wv[i], wv[i]), __fmul_rn(d, d));
  }
  uint32_t flag[B / 32];
  for (int q = 0; q < B / 32; ++q) flag[q] = 0;
  for (int t = 0; t < kt; ++t) {  // k passes of "largest importance not yet taken, lowest channel on ties"
    int best = -1;
    float bv = -1.0f;
    for (int i = 0; i < B; ++i) {
      const bool taken = (flag[i >> 5] >> (i & 31)) & 1u;
      if (!taken && imp[i] > bv) {
        bv = imp[i];
        best = i;
      }
    }
    if (best >= 0) flag[best >> 5] |= 1u << (best & 31);
  }
  float a_hi = 0.0f, a_lo = 0.0f;
  for (int i = 0; i < B; ++i) {
    const float a = fabsf(wv[i]);
    if ((flag[i >> 5] >> (i & 31)) & 1u) a_hi = fmaxf(a_hi, a);
    else a_lo = fmaxf(a_lo, a);
  }
  const float inv_hi = a_hi != 0.0f ? __fdiv_rn(q_hi, a_hi) : 0.0f;
  const float inv_lo = a_lo != 0.0f ? __fdiv_rn(q_lo, a_lo) : 0.0f;
  s_hi[idx] = a_hi != 0.0f ? __fdiv_rn(a_hi, q_hi) : 1.0f;
  s_lo[idx] = a_lo != 0.0f ? __fdiv_rn(a_lo, q_lo) : 1.0f;
  uint8_t* ldst = lo + n * (K / 2) + static_cast<int64_t>(g) * (B / 2);
  int8_t* hdst = hi_val + idx * kt;
  int nh = 0;
  const int iq_hi = static_cast<int>(q_hi), iq_lo = static_cast<int>(q_lo);
  for (int i = 0; i < B; i += 2) {
    uint32_t byte = 0;
    for (int e = 0; e < 2; ++e) {
      int code;
      if ((flag[(i + e) >> 5] >> ((i + e) & 31)) & 1u) {
        const int c = min(max(rne_code(wv[i + e], inv_hi), -iq_hi), iq_hi);
        if (nh < kt) hdst[nh] = static_cast<int8_t>(c);
        ++nh;
        code = v_mask;
      } else {
        code = min(max(rne_code(wv[i + e], inv_lo), -iq_lo), iq_lo);
      }
      byte |= static_cast<uint32_t>(code & 0xF) << (4 * e);
    }
    ldst[i / 2] = static_cast<uint8_t>(byte);
  }
}

// ---- offline: compute-ready image of the weights: the low part with zeros at the high positions, and the high
// part as a zero-padded INT8 matrix in the byte order the widened low part unfolds to (per 8 channels: the even
// channels, then the odd ones).  One thread per 32 channels. ----
__global__ __launch_bounds__(256) void wsq_prepack_kernel(int N, int K, int B, int kt, int vm_nibble,
                                                          const uint8_t* __restrict__ lo, const int8_t* __restrict__ hi_val,
                                                          uint8_t* __restrict__ lo_clean, int8_t* __restrict__ hi_dense) {
  const int wpr = K / 32;
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= static_cast<int64_t>(N) * wpr) return;
  const int64_t n = idx / wpr;
  const int wg = static_cast<int>(idx - n * wpr);
  const int bank = wg / (B / 32);
  const uint8_t* row = lo + n * (K / 2);
  int rank = 0;  // high weights of the bank before this word
  for (int ch = bank * B; ch < wg * 32; ++ch) rank += ((row[ch >> 1] >> ((ch & 1) * 4)) & 0xF) == vm_nibble;
  const int8_t* hv = hi_val + (n * (K / B) + bank) * kt;
  uint32_t clean[4] = {0, 0, 0, 0};
  int8_t dense[32];
  for (int i = 0; i < 32; ++i) dense[i] = 0;
  for (int i = 0; i < 32; ++i) {
    const int ch = wg * 32 + i;
    const int nib = (row[ch >> 1] >> ((ch & 1) * 4)) & 0xF;
    if (nib == vm_nibble) {
      const int pos = (i & ~7) | ((i & 1) << 2) | ((i & 7) >> 1);
      dense[pos] = rank < kt ? hv[rank] : 0;
      ++rank;
    } else {
      clean[i >> 3] |= static_cast<uint32_t>(nib) << (4 * (i & 7));
    }
  }
  *reinterpret_cast<uint4*>(lo_clean + n * (K / 2) + static_cast<int64_t>(wg) * 16) = make_uint4(clean[0], clean[1], clean[2], clean[3]);
  int8_t* hd = hi_dense + n * K + static_cast<int64_t>(wg) * 32;
  for (int i = 0; i < 32; ++i) hd[i] = dense[i];
}

// ---- run time: plain per-token symmetric quantisation of the activations (Section 4.1: the operand that is not
// in SQ-format is plain INTy), codes written in the byte order of the weight images.  One workgroup per row; a row of up
// to 2048 IT channels is read once and kept in registers between its maximum and its codes (IT = 0: read twice).  Bound
// by HBM, 3 bytes per element ([4096,4096] 11.4 us; read twice it took 20.9 us). ----
template <int IT>
__global__ __launch_bounds__(256) void quantize_act_kernel(const uint16_t* __restrict__ x, int64_t ldx, int K, float q,
                                                           int8_t* __restrict__ a8, float* __restrict__ a_scale) {
  __shared__ uint32_t wave_max[4];
  const int64_t m = blockIdx.x;
  const uint16_t* row = x + m * ldx;
  const int tid = threadIdx.x, n = K / 8;
  v4u keep[IT > 0 ? IT : 1];
  uint32_t mx = 0;
  auto piece_max = [&](const v4u& v) {
    for (int e = 0; e < 4; ++e) mx = max(mx, max(v[e] & 0x7FFFu, (v[e] >> 16) & 0x7FFFu));
  };
  if constexpr (IT > 0) {
#pragma unroll
    for (int i = 0; i < IT; ++i) keep[i] = *reinterpret_cast<const v4u*>(row + min(i * 256 + tid, n - 1) * 8);
#pragma unroll
    for (int i = 0; i < IT; ++i) piece_max(keep[i]);
  } else {
    for (int c = tid; c < n; c += 256) piece_max(*reinterpret_cast<const v4u*>(row + c * 8));
  }
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) mx = max(mx, static_cast<uint32_t>(__shfl_xor(static_cast<int>(mx), off, 64)));
  if ((tid & 63) == 0) wave_max[tid >> 6] = mx;
  __syncthreads();
  const uint32_t am = max(max(wave_max[0], wave_max[1]), max(wave_max[2], wave_max[3]));
  const float amax = __uint_as_float(am << 16);
  const float inv = am ? __fdiv_rn(q, amax) : 0.0f;
  if (tid == 0) a_scale[m] = am ? __fdiv_rn(amax, q) : 1.0f;
  auto piece_codes = [&](const v4u& v, int c) {
    uint32_t ev = 0, od = 0;  // codes of the even / odd channels of the group, the first one ends in the low byte
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x0 = __fmul_rn(__uint_as_float(v[e] << 16), inv), x1 = __fmul_rn(__uint_as_float(v[e] & 0xFFFF0000u), inv);
      ev = __builtin_amdgcn_alignbit(__float_as_uint(__fadd_rn(__builtin_amdgcn_fmed3f(x0, -q, q), kMagic)), ev, 8);
      od = __builtin_amdgcn_alignbit(__float_as_uint(__fadd_rn(__builtin_amdgcn_fmed3f(x1, -q, q), kMagic)), od, 8);
    }
    *reinterpret_cast<v2u*>(a8 + m * K + c * 8) = v2u{ev, od};
  };
  if constexpr (IT > 0) {
#pragma unroll
    for (int i = 0; i < IT; ++i)
      if (i * 256 + tid < n) piece_codes(keep[i], i * 256 + tid);
  } else {
    for (int c = tid; c < n; c += 256) piece_codes(*reinterpret_cast<const v4u*>(row + c * 8), c);
  }
}

__device__ __forceinline__ v4i widen_half(const v4u p, int s) {
  const unsigned a = p[2 * s], b = p[2 * s + 1];
  return v4i{static_cast<int>((a << 4) & 0xF0F0F0F0u), static_cast<int>(a & 0xF0F0F0F0u),
             static_cast<int>((b << 4) & 0xF0F0F0F0u), static_cast<int>(b & 0xF0F0F0F0u)};
}

struct WsqGemmArgs {
  int M, N, K, G;
  const int8_t* a8;        // [M, K] activation codes
  const float* a_scale;    // [M]
  const uint8_t* lo_clean; // [N, K/2]
  const int8_t* hi_dense;  // [N, K]
  const float* s_lo;       // [N, G]
  const float* s_hi;
  void* y;
  int64_t ldy;
  int out_bf16;
  int32_t* acc_lo_dbg;     // optional [M, N, G]
  int32_t* acc_hi_dbg;
};

// The per-bank products themselves (tests): 64 tokens x 64 output channels per workgroup, four waves of 32 x 32; one
// bank per trip, single-buffered.
template <int B>
__global__ __launch_bounds__(256) void wsq_gemm_kernel(WsqGemmArgs g) {
  __shared__ __attribute__((aligned(16))) char s_a[64 * B];       // activation codes of the bank
  __shared__ __attribute__((aligned(16))) char s_wl[64 * (B / 2)];  // packed low weights
  __shared__ __attribute__((aligned(16))) char s_wh[64 * B];      // INT8 high weights
  __shared__ float s_sl[64], s_sh[64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int r = lane & 31, h = lane >> 5;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  float f[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) f[q] = 0.0f;

  for (int bank = 0; bank < g.G; ++bank) {
    // ---- stage the bank's operands (rows past the edge re-read the last row; never stored) ----
    for (int c = tid; c < 64 * B / 16; c += 256) {
      const int row = c / (B / 16), ch = c % (B / 16);
      *reinterpret_cast<v4u*>(s_a + row * B + ch * 16) =
          *reinterpret_cast<const v4u*>(g.a8 + static_cast<int64_t>(min(m0 + row, g.M - 1)) * g.K + bank * B + ch * 16);
      *reinterpret_cast<v4u*>(s_wh + row * B + ch * 16) =
          *reinterpret_cast<const v4u*>(g.hi_dense + static_cast<int64_t>(min(n0 + row, g.N - 1)) * g.K + bank * B + ch * 16);
    }
    for (int c = tid; c < 64 * B / 32; c += 256) {
      const int row = c / (B / 32), ch = c % (B / 32);
      *reinterpret_cast<v4u*>(s_wl + row * (B / 2) + ch * 16) =
          *reinterpret_cast<const v4u*>(g.lo_clean + static_cast<int64_t>(min(n0 + row, g.N - 1)) * (g.K / 2) + bank * (B / 2) + ch * 16);
    }
    if (tid < 64) {
      const int64_t n = min(n0 + tid, g.N - 1);
      s_sl[tid] = g.s_lo[n * g.G + bank];
      s_sh[tid] = g.s_hi[n * g.G + bank];
    }
    __syncthreads();

    // ---- the bank's two integer products (exact) ----
    v16i acc_lo, acc_hi;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      acc_lo[q] = 0;
      acc_hi[q] = 0;
    }
#pragma unroll
    for (int kb = 0; kb < B / 64; ++kb) {
      const v4u wl = *reinterpret_cast<const v4u*>(s_wl + (32 * wn + r) * (B / 2) + kb * 32 + h * 16);
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const v4i a16 = *reinterpret_cast<const v4i*>(s_a + (32 * wm + r) * B + kb * 64 + (2 * h + s) * 16);
        const v4i wh = *reinterpret_cast<const v4i*>(s_wh + (32 * wn + r) * B + kb * 64 + (2 * h + s) * 16);
        acc_lo = __builtin_amdgcn_mfma_i32_32x32x32_i8(a16, widen_half(wl, s), acc_lo, 0, 0, 0);
        acc_hi = __builtin_amdgcn_mfma_i32_32x32x32_i8(a16, wh, acc_hi, 0, 0, 0);
      }
    }
    // ---- fold into the fp32 accumulator, in the layer's fixed order ----
    const float sl = s_sl[32 * wn + r], sh = s_sh[32 * wn + r];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int alo = acc_lo[q] >> 4;  // the widened low weights carry a factor 16
      float t = __fmul_rn(static_cast<float>(alo), sl);
      t = __fmaf_rn(static_cast<float>(acc_hi[q]), sh, t);
      f[q] = __fadd_rn(f[q], t);
      if (g.acc_lo_dbg || g.acc_hi_dbg) {
        const int m = m0 + 32 * wm + 8 * (q >> 2) + 4 * h + (q & 3), n = n0 + 32 * wn + r;
        if (m < g.M && n < g.N) {
          const int64_t o = (static_cast<int64_t>(m) * g.N + n) * g.G + bank;
          if (g.acc_lo_dbg) g.acc_lo_dbg[o] = alo;
          if (g.acc_hi_dbg) g.acc_hi_dbg[o] = acc_hi[q];
        }
      }
    }
    __syncthreads();  // the tiles are overwritten by the next bank
  }
  // ---- epilogue ----
  const int n = n0 + 32 * wn + r;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int m = m0 + 32 * wm + 8 * (q >> 2) + 4 * h + (q & 3);
    if (m < g.M && n < g.N) {
      const float y = __fmul_rn(f[q], g.a_scale[m]);
      const int64_t o = static_cast<int64_t>(m) * g.ldy + n;
      if (g.out_bf16) reinterpret_cast<uint16_t*>(g.y)[o] = f32_to_bf16_rne(y);
      else reinterpret_cast<float*>(g.y)[o] = y;
    }
  }
}

// ---- the throughput kernel ----
// 32 MW tokens x 128 output channels per workgroup, 2 MW waves of 32 x 64.  The operands of a bank (BPB stages of 64
// channels: activation codes, INT8 high weights, packed low weights; and the bank's scales) are copied into a ring of LDS
// stages by LDS-direct loads, R - 1 banks ahead, rows XOR-swizzled as in the activation-SQ kernel.  A wave multiplies one
// 32 x 32 tile of the bank (4 * BPB matrix instructions into 32 integer registers) and folds it into its fp32
// accumulators (5 vector instructions per register) before it starts on the next tile: with so few registers four waves
// share a SIMD, and one wave's fold runs under the others' matrix instructions.  That fold bounds the kernel: 1280 cycles
// per 64 x 64 outputs and bank against 512 * BPB of matrix instructions.  With four waves of 64 x 64 per workgroup (all
// four tiles' integer registers live, two waves per SIMD) the two hardly overlapped:
// [4096,4096] x [22016,4096] 1241 -> 1106 us with banks of 64, 1012 -> 868 us with banks of 128 (whole calls, in turn on one
// card); [300,4096] x [4096,4096] 96 -> 66 us; [8,4096] x [12288,4096] 106 -> 66 us (the single-buffered kernel ran there).
// PAIR (banks of 128): the 128-token tile with the bank's scales read from memory by the lanes, before they copy the next bank
// (a later read would wait for the copies).  The 2 KB of LDS that this saves let two workgroups share a compute unit: with one,
// nothing ran under a workgroup's start and epilogue, and shapes of several rounds had become up to 15 % slower than with the
// 64 x 64 waves ([2566,640] x [9054,640] 92 -> 106 us, now 84 us).
// TINY: low scales below 2^-122 count, too (see w2_exact).  Calls of up to 64 tokens always took them; keeping the least scale
// costs them 0.7 %.
template <int BPB_, int MW_, bool PAIR = false, bool TINY_ = false>
struct W2 {
  static constexpr bool TINY = TINY_;
  static constexpr int BPB = BPB_, MW = MW_;
  static constexpr int BM = 32 * MW, THREADS = 128 * MW;
  static constexpr int A = 0, WH = BM * 64, WL = WH + 8192, STAGE = WL + 4096;  // a 64-channel stage
  static constexpr bool SC_LDS = !PAIR;
  static constexpr int SC = BPB * STAGE, BANK = SC + (SC_LDS ? 1024 : 0);      // the bank's scales: 128 low, 128 high
  static constexpr int FIT = (MW == 4 ? 80 : 160) * 1024 / BANK;  // two workgroups per compute unit, or one
  static constexpr int R = FIT > 4 ? 4 : (FIT < 2 ? 2 : FIT);
  static constexpr int EPI = 2 * MW * 32 * (64 * 4 + 16);  // the epilogue's buffers
  static constexpr int LDS_BYTES = R * BANK > EPI ? R * BANK : EPI;
  static_assert(LDS_BYTES <= (PAIR ? 80 : 160) * 1024, "LDS");
};

__device__ __forceinline__ int w2_off2(int row, int c) { return (row << 5) + (((c ^ (row >> 3)) & 1) << 4); }  // 32-byte rows

template <int N>
__device__ __forceinline__ void w2_wait() {  // at most N vector-memory operations outstanding, LDS reads drained, barrier
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (0 << 8) | ((N >> 4) << 14));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

struct Wsq2Args {
  int M, N, K, G, Npad;
  const int8_t* a8;
  const float* a_scale;
  const uint8_t* lo_clean;
  const int8_t* hi_dense;
  const float* s_lo_t;  // [G, Npad]
  const float* s_hi_t;
  const float* s_lo;    // [N, G]
  void* y;
  int64_t ldy;
  int out_bf16;
};

template <typename OutT>
__device__ __forceinline__ void w2_epilogue(const Wsq2Args& g, char* tb, const float (&f)[2][16], int m0, int n0, int lane) {
  // the wave's 32 x 64 outputs through LDS, then 16 bytes per lane
  constexpr int ESZ = sizeof(OutT), ROW = 64 * ESZ + 16, PER16 = 16 / ESZ, CHUNKS = 64 / PER16, ROWS = 64 / CHUNKS;
  const int r = lane & 31, h = lane >> 5;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int rl = 8 * (q >> 2) + 4 * h + (q & 3);
    const float sa = g.a_scale[min(m0 + rl, g.M - 1)];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float y = __fmul_rn(f[j][q], sa);
      OutT* dst = reinterpret_cast<OutT*>(tb + rl * ROW) + j * 32 + r;
      if constexpr (ESZ == 2) *dst = gemm::bf16_rne(y);
      else *dst = y;
    }
  }
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((15) | (7 << 4) | (0 << 8) | (3 << 14));  // lgkmcnt(0): the buffer is the wave's own
  asm volatile("" ::: "memory");
  const bool vec_ok = (g.ldy % PER16) == 0;
#pragma unroll
  for (int p0 = 0; p0 < 32; p0 += ROWS) {
    const int rl = p0 + lane / CHUNKS, ch = lane % CHUNKS, m = m0 + rl, n = n0 + ch * PER16;
    if (m < g.M && n < g.N) {
      OutT* dst = reinterpret_cast<OutT*>(g.y) + static_cast<int64_t>(m) * g.ldy + n;
      if (vec_ok && n + PER16 <= g.N) {
        *reinterpret_cast<v4u*>(dst) = *reinterpret_cast<const v4u*>(tb + rl * ROW + ch * 16);
      } else {
        const OutT* src = reinterpret_cast<const OutT*>(tb + rl * ROW + ch * 16);
        for (int q = 0; q < PER16 && n + q < g.N; ++q) dst[q] = src[q];
      }
    }
  }
}

// A wave's 32 x 64 sums from the scales as they are given: the transposed low scales are divided by 16, which loses bits of
// those below 2^-122.  Straight from memory, for the rare tile that has such a scale.
template <int BPB>
__device__ __forceinline__ void w2_exact(const Wsq2Args& g, float (&f)[2][16], int m0, int n0, int lane) {
  const int r = lane & 31, h = lane >> 5;
  const int8_t* a8 = g.a8 + static_cast<int64_t>(min(m0 + r, g.M - 1)) * g.K;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int64_t n = min(n0 + 32 * j + r, g.N - 1);
    const uint8_t* wl = g.lo_clean + n * (g.K / 2);
    const int8_t* wh = g.hi_dense + n * g.K;
#pragma unroll
    for (int q = 0; q < 16; ++q) f[j][q] = 0.0f;
    for (int bank = 0; bank < g.G; ++bank) {
      v16i acc_lo = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}, acc_hi = acc_lo;
      for (int k = bank * BPB * 64; k < (bank + 1) * BPB * 64; k += 64) {
        const v4u l = *reinterpret_cast<const v4u*>(wl + k / 2 + 16 * h);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const v4i a = *reinterpret_cast<const v4i*>(a8 + k + 16 * (2 * h + s));
          acc_lo = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, widen_half(l, s), acc_lo, 0, 0, 0);
          acc_hi = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, *reinterpret_cast<const v4i*>(wh + k + 16 * (2 * h + s)), acc_hi, 0, 0, 0);
        }
      }
      const float sl = g.s_lo[n * g.G + bank], sh = g.s_hi_t[static_cast<int64_t>(bank) * g.Npad + n];
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const float t = __fmul_rn(static_cast<float>(acc_lo[q] >> 4), sl);
        f[j][q] = __fadd_rn(f[j][q], __fmaf_rn(static_cast<float>(acc_hi[q]), sh, t));
      }
    }
  }
}

template <typename C>
__global__ __launch_bounds__(C::THREADS, 4) void wsq_gemm2_kernel(Wsq2Args g) {
  constexpr int BPB = C::BPB, MW = C::MW;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int r = lane & 31, h = lane >> 5;
  int tm, tn;
  gemm::tile_of_block(blockIdx.x, (g.M + C::BM - 1) / C::BM, (g.N + 127) / 128, tm, tn);
  if (tm < 0) return;
  const int m0 = tm * C::BM, n0 = tn * 128;

  // per-lane sources of the copies of one stage (at k = 0).  Every wave copies its share of the activations; the weights
  // and the scales are dealt to some of them.
  constexpr int WL0 = MW == 4 ? 0 : 8, WSC = WL0 + 4;  // first wave of the low weights (four of them), wave of the scales
  const bool has_wh = MW == 4 || wave < 8, has_wl = wave >= WL0 && wave < WL0 + 4, has_sc = C::SC_LDS && wave == WSC;
  const char *pa, *pwh, *pwl, *psc;
  {
    const int row = tid >> 2, c = ((tid & 3) ^ (row >> 2)) & 3;
    pa = reinterpret_cast<const char*>(g.a8) + static_cast<int64_t>(min(m0 + row, g.M - 1)) * g.K + c * 16;
    const int rowh = (tid & 511) >> 2;
    pwh = reinterpret_cast<const char*>(g.hi_dense) + static_cast<int64_t>(min(n0 + rowh, g.N - 1)) * g.K + c * 16;
    const int row2 = (tid & 255) >> 1, c2 = ((tid & 1) ^ (row2 >> 3)) & 1;
    pwl = reinterpret_cast<const char*>(g.lo_clean) + static_cast<int64_t>(min(n0 + row2, g.N - 1)) * (g.K / 2) + c2 * 16;
    // lanes 0-31 fetch the low scales of the workgroup's 128 channels, lanes 32-63 the high ones
    psc = reinterpret_cast<const char*>(lane < 32 ? g.s_lo_t : g.s_hi_t) + (static_cast<int64_t>(n0) + (lane & 31) * 4) * 4;
  }
  auto issue = [&](int bank) {
    char* base = lds + (bank % C::R) * C::BANK;
#pragma unroll
    for (int b = 0; b < BPB; ++b) {
      const int step = bank * BPB + b;
      char* st = base + b * C::STAGE;
      __builtin_amdgcn_global_load_lds(pa + step * 64, (lds_ptr_t)(st + C::A + 1024 * wave), 16, 0, 0);
      if (has_wh) __builtin_amdgcn_global_load_lds(pwh + step * 64, (lds_ptr_t)(st + C::WH + 1024 * wave), 16, 0, 0);
      if (has_wl) __builtin_amdgcn_global_load_lds(pwl + step * 32, (lds_ptr_t)(st + C::WL + 1024 * (wave - WL0)), 16, 0, 0);
    }
    if (has_sc) {
      const char* src = psc + static_cast<int64_t>(bank) * g.Npad * 4;
      __builtin_amdgcn_global_load_lds(src, (lds_ptr_t)(base + C::SC), 16, 0, 0);
    }
  };
  const int per_bank = BPB * (1 + has_wh + has_wl) + has_sc;  // copies of this wave per bank: 1 ... 6
#pragma unroll
  for (int b = 0; b < C::R - 1; ++b)
    if (b < g.G) issue(b);

  float f[2][16];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q = 0; q < 16; ++q) f[j][q] = 0.0f;
  const v16i zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  float least[2] = {1.0f, 1.0f};  // TINY: of the lane's low scales

  for (int bank = 0; bank < g.G; ++bank) {
    // this wave's copies of the bank have landed when at most those of the R - 2 banks after it are in flight
    if (C::R == 2 || bank + C::R - 2 >= g.G) w2_wait<0>();
    else if (per_bank >= 3) w2_wait<(C::R - 2) * 3>();
    else if (per_bank == 2) w2_wait<(C::R - 2) * 2>();
    else w2_wait<C::R - 2>();
    // the stages of bank - 1 are free: every wave has read them for the last time before this barrier
    float sl[2], sh[2];
    if constexpr (!C::SC_LDS) {  // before the copies of the next bank, which the wait for them then leaves in flight
      const int64_t o = static_cast<int64_t>(bank) * g.Npad + n0 + 64 * wn + r;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        sl[j] = g.s_lo_t[o + 32 * j];
        sh[j] = g.s_hi_t[o + 32 * j];
      }
    }
    if (bank + C::R - 1 < g.G) issue(bank + C::R - 1);
    const char* st0 = lds + (bank % C::R) * C::BANK;
    const float* sc = reinterpret_cast<const float*>(st0 + C::SC) + 64 * wn + r;
    v4i a[BPB][2];
#pragma unroll
    for (int b = 0; b < BPB; ++b)
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
        a[b][s2] = *reinterpret_cast<const v4i*>(st0 + b * C::STAGE + C::A + gemm::off4(32 * wm + r, 2 * h + s2));
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      v16i acc_lo = zero, acc_hi = zero;
      if constexpr (C::SC_LDS) {
        sl[j] = sc[32 * j];
        sh[j] = sc[128 + 32 * j];
      }
#pragma unroll
      for (int b = 0; b < BPB; ++b) {
        const char* st = st0 + b * C::STAGE;
        const v4u wl = *reinterpret_cast<const v4u*>(st + C::WL + w2_off2(64 * wn + 32 * j + r, h));
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          const v4i wh = *reinterpret_cast<const v4i*>(st + C::WH + gemm::off4(64 * wn + 32 * j + r, 2 * h + s2));
          acc_lo = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[b][s2], widen_half(wl, s2), acc_lo, 0, 0, 0);
          acc_hi = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[b][s2], wh, acc_hi, 0, 0, 0);
        }
      }
      if constexpr (C::TINY) least[j] = fminf(least[j], fabsf(sl[j]));
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        // the widened low weights carry a factor 16, which the transposed low scales carry inverted (sl is
        // s_lo / 16: float(16 a) * (s / 16) is float(a) * s bit for bit while s / 16 is a normal number)
        float t = __fmul_rn(static_cast<float>(acc_lo[q]), sl[j]);
        t = __fmaf_rn(static_cast<float>(acc_hi[q]), sh[j], t);
        f[j][q] = __fadd_rn(f[j][q], t);
      }
    }
  }
  if constexpr (C::TINY) {
    const int n = n0 + 64 * wn + r;  // (beyond N the scales are zero)
    if (__any((least[0] < 0x1p-126f && n < g.N) || (least[1] < 0x1p-126f && n + 32 < g.N)))
      w2_exact<BPB>(g, f, m0 + 32 * wm, n0 + 64 * wn, lane);
  }
  __syncthreads();  // the stages are free: y = f * s_a[m]
  char* tb = lds + wave * (32 * (64 * 4 + 16));
  if (g.out_bf16) w2_epilogue<uint16_t>(g, tb, f, m0 + 32 * wm, n0 + 64 * wn, lane);
  else w2_epilogue<float>(g, tb, f, m0 + 32 * wm, n0 + 64 * wn, lane);
}

// scales [N, G] -> [G, Npad] (zero beyond N), so that a bank's scales of 128 consecutive channels are contiguous;
// the low scales are stored divided by 16 (exact for every scale above 2^-122)
__global__ __launch_bounds__(256) void wsq_scales_t_kernel(int N, int G, int Npad, const float* __restrict__ s_lo,
                                                           const float* __restrict__ s_hi, float* __restrict__ lo_t,
                                                           float* __restrict__ hi_t) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= static_cast<int64_t>(G) * Npad) return;
  const int gq = static_cast<int>(idx / Npad), n = static_cast<int>(idx - static_cast<int64_t>(gq) * Npad);
  lo_t[idx] = n < N ? s_lo[static_cast<int64_t>(n) * G + gq] * 0.0625f : 0.0f;  // / 16: see the fold of wsq_gemm2_kernel
  hi_t[idx] = n < N ? s_hi[static_cast<int64_t>(n) * G + gq] : 0.0f;
}

}  // namespace

int init_wsq_kernels() {
  hipError_t e = hipSuccess;
#define X(...)                                                                                           \
  if (e == hipSuccess)                                                                                   \
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(wsq_gemm2_kernel<W2<__VA_ARGS__>>),            \
                            hipFuncAttributeMaxDynamicSharedMemorySize, W2<__VA_ARGS__>::LDS_BYTES);
  X(1, 4) X(1, 8) X(2, 4) X(2, 8) X(2, 4, true)
  X(1, 4, false, true) X(2, 4, false, true) X(2, 4, true, true)
#undef X
  return e == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}

template <typename C>
void launch_wsq2(const Wsq2Args& a, hipStream_t st) {
  const int tiles = ((a.N + 127) / 128) * ((a.M + C::BM - 1) / C::BM);
  hipLaunchKernelGGL(wsq_gemm2_kernel<C>, dim3((tiles + 7) / 8 * 8), dim3(C::THREADS), C::LDS_BYTES, st, a);
}

int launch_wsq_encode(const sq_params& p, const uint16_t* w, int64_t ldw, const float* hinv, const sq_wsq& out, hipStream_t st) {
  const int G = p.K / p.bank;
  const int64_t groups = static_cast<int64_t>(p.N) * G;
  const unsigned blocks = static_cast<unsigned>((groups + 63) / 64);
  const float q_hi = code_max(p.h_high, 8), q_lo = code_max(p.h_low, 4);
  const int v_mask = -(1 << ((p.h_low ? p.h_low : 4) - 1));
  if (p.bank == 64)
    hipLaunchKernelGGL(wsq_encode_kernel<64>, dim3(blocks), dim3(64), 0, st, w, ldw, p.N, p.K, p.topk, hinv, q_hi, q_lo, v_mask,
                       out.lo, out.hi_val, out.scale_lo, out.scale_hi);
  else
    hipLaunchKernelGGL(wsq_encode_kernel<128>, dim3(blocks), dim3(64), 0, st, w, ldw, p.N, p.K, p.topk, hinv, q_hi, q_lo, v_mask,
                       out.lo, out.hi_val, out.scale_lo, out.scale_hi);
  return hipGetLastError() == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}

int launch_wsq_prepack(const sq_params& p, const sq_wsq& w, uint8_t* lo_clean, int8_t* hi_dense, float* s_lo_t, float* s_hi_t,
                       hipStream_t st) {
  const int64_t total = static_cast<int64_t>(p.N) * (p.K / 32);
  const int vm = (-(1 << ((p.h_low ? p.h_low : 4) - 1))) & 0xF;
  hipLaunchKernelGGL(wsq_prepack_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, st, p.N, p.K, p.bank,
                     p.topk, vm, w.lo, w.hi_val, lo_clean, hi_dense);
  if (hipGetLastError() != hipSuccess) return SQ_ERR_LAUNCH;
  const int G = p.K / p.bank, Npad = (p.N + 127) / 128 * 128;
  const int64_t n_sc = static_cast<int64_t>(G) * Npad;
  hipLaunchKernelGGL(wsq_scales_t_kernel, dim3(static_cast<unsigned>((n_sc + 255) / 256)), dim3(256), 0, st, p.N, G, Npad,
                     w.scale_lo, w.scale_hi, s_lo_t, s_hi_t);
  return hipGetLastError() == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}

int launch_quantize_act(const sq_params& p, const uint16_t* x, int64_t ldx, int bits, int8_t* a8, float* a_scale, hipStream_t st) {
#define X(IT) hipLaunchKernelGGL(quantize_act_kernel<IT>, dim3(p.M), dim3(256), 0, st, x, ldx, p.K, code_max(bits, 8), a8, a_scale)
  if (p.K <= 4096) X(2);
  else if (p.K <= 8192) X(4);
  else if (p.K <= 16384) X(8);
  else X(0);
#undef X
  return hipGetLastError() == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}

int launch_wsq_gemm(const sq_params& p, const int8_t* a8, const float* a_scale, const sq_wsq& w, const uint8_t* lo_clean,
                    const int8_t* hi_dense, const float* s_lo_t, const float* s_hi_t, void* y, int64_t ldy,
                    int32_t* acc_lo_dbg, int32_t* acc_hi_dbg, hipStream_t st) {
  if (!acc_lo_dbg && !acc_hi_dbg) {  // the kernel below is for dumping the per-bank products
    Wsq2Args a;
    a.M = p.M;
    a.N = p.N;
    a.K = p.K;
    a.G = p.K / p.bank;
    a.Npad = (p.N + 127) / 128 * 128;
    a.a8 = a8;
    a.a_scale = a_scale;
    a.lo_clean = lo_clean;
    a.hi_dense = hi_dense;
    a.s_lo_t = s_lo_t;
    a.s_hi_t = s_hi_t;
    a.s_lo = w.scale_lo;
    a.y = y;
    a.ldy = ldy;
    a.out_bf16 = p.out_dtype == SQ_OUT_BF16;
    // 256 tokens per workgroup (30 % less operand traffic; it takes a compute unit alone) or 128, by the rounds that the 256
    // compute units make.  Banks of 64: two of the 128-token tiles share a unit, so that one's start and epilogue run under the
    // other's banks: 128 tokens (1106 against 1142 us at [4096,4096] x [22016,4096], 302 against 361 us at [4487,640] x
    // [21543,640], 59 against 103 us at [600,2048] x [11008,2048]), unless the tall tiles make one round that is 15/16 full
    // (22.5 against 24.3 us at [398,128] x [16251,128], 101 against 103 us at [716,3456] x [10406,3456]).
    // Banks of 128: up to one round of 128-token tiles the scales come through LDS (111 against 135 us at
    // [656,9344] x [369,9344] with the lanes reading them); beyond that pairs of them share a unit (126 against 147 us at
    // [1505,768] x [23028,768], 88 against 101 us at [1100,4096] x [6912,4096]), unless the tall tiles make one round (178 us
    // against 196 us for pairs at [493,9472] x [13810,9472]) or 7/8 full ones of long rows (172 against 179 us at [4096,4096] x
    // [4096,4096]; 554 against 539 us at [4009,1408] x [28591,1408], 315 against 348 us where the last is half empty, at
    // [1610,5632] x [12399,5632]).
    const int64_t cols = (p.N + 127) / 128, short_tiles = cols * ((p.M + 127) / 128), tall_tiles = cols * ((p.M + 255) / 256);
    const int64_t tall_rounds = (tall_tiles + 255) / 256;
    if (p.M <= 64) {
      if (p.bank == 64) launch_wsq2<W2<1, 4, false, true>>(a, st);
      else short_tiles <= 256 ? launch_wsq2<W2<2, 4, false, true>>(a, st) : launch_wsq2<W2<2, 4, true, true>>(a, st);
    } else if (p.bank == 64) {
      tall_rounds == 1 && short_tiles >= 480 ? launch_wsq2<W2<1, 8>>(a, st) : launch_wsq2<W2<1, 4>>(a, st);
    } else if (short_tiles <= 256) {
      launch_wsq2<W2<2, 4>>(a, st);
    } else {
      const bool tall = tall_rounds == 1 ? p.K >= 640 : p.K >= 2048 && 448 * tall_rounds <= short_tiles;
      tall ? launch_wsq2<W2<2, 8>>(a, st) : launch_wsq2<W2<2, 4, true>>(a, st);
    }
    return hipGetLastError() == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
  }
  WsqGemmArgs g;
  g.M = p.M;
  g.N = p.N;
  g.K = p.K;
  g.G = p.K / p.bank;
  g.a8 = a8;
  g.a_scale = a_scale;
  g.lo_clean = lo_clean;
  g.hi_dense = hi_dense;
  g.s_lo = w.scale_lo;
  g.s_hi = w.scale_hi;
  g.y = y;
  g.ldy = ldy;
  g.out_bf16 = p.out_dtype == SQ_OUT_BF16;
  g.acc_lo_dbg = acc_lo_dbg;
  g.acc_hi_dbg = acc_hi_dbg;
  const dim3 grid((p.N + 63) / 64, (p.M + 63) / 64);
  if (p.bank == 64) hipLaunchKernelGGL(wsq_gemm_kernel<64>, grid, dim3(256), 0, st, g);
  else hipLaunchKernelGGL(wsq_gemm_kernel<128>, grid, dim3(256), 0, st, g);
  return hipGetLastError() == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}

}  // namespace sq
