// sq_encode, dynamic rule, for few banks (gfx950): bf16 activations -> SQ-format, the same results as the other encoders.
//
// With one lane per bank a short call is one wave per SIMD that works through 1500 (bank 64) or 4000 (bank 128) dependent
// vector instructions, about 2 ns each, while most of the chip idles.  Here LPB neighbouring lanes share a bank: each
// selects the k largest of its own channels (the same comparator networks), the sorted lists are merged across the lanes
// (quad permutations; max(a_i, b_{k-1-i}) keeps the k largest of two descending lists, so that all lanes of the bank end
// up with the same set), and each lane quantises and stores its own channels.  A workgroup is one token row, or, where a
// row has at most 32 lanes, one wave of several rows (with a wave per row most lanes idled and the wave took as long:
// [1905,192] b = 64, k = 32 20.1 -> 6.2 us; with a lane per bank 7.7 us).
// Bounded by that chain (about 650 instructions at bank 64, k = 8) and by launch and memory latency:
// [1,8192] 5.7 -> 3.9 us, [64,8192] 6.3 -> 4.3 us, [128,8192] bank 128, k = 32 14.4 -> 7.5 us.
#include "sq_encode_common.h"

namespace sq {
namespace {

using namespace enc;

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

constexpr int kThreads = 512;

struct FewEncArgs {
  const uint16_t* x;
  int64_t ldx;
  int M, K, G;
  int lg_span;        // SHARED: lanes of a row, a power of two up to 32
  uint8_t* d_lo;
  int8_t* hi_val;
  uint32_t* mask;
  float* s_lo;
  float* s_hi;
  int8_t* image;     // hi_dense (two scales) or the combined INT8 operand (TIED); may be null
  float q_hi, q_lo;
};

// lane ^ 1, lane ^ 2 (inside four lanes)
template <int X>
__device__ __forceinline__ uint32_t quad_xor(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), X == 1 ? 0xB1 : 0x4E, 0xF, 0xF, true));
}
__device__ __forceinline__ uint32_t pk_max_u16(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
// maximum over every 2^lg lanes (lg = 1 ... 6), both halves of the word for themselves
__device__ __forceinline__ uint32_t span_pk_max(uint32_t v, int lg) {
  v = pk_max_u16(v, quad_xor<1>(v));
  if (lg > 1) v = pk_max_u16(v, quad_xor<2>(v));
  if (lg > 2) v = pk_max_u16(v, static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), 0x141, 0xF, 0xF, true)));  // row_half_mirror
  if (lg > 3) v = pk_max_u16(v, static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), 0x140, 0xF, 0xF, true)));  // row_mirror
  if (lg > 4) v = pk_max_u16(v, static_cast<uint32_t>(__shfl_xor(static_cast<int>(v), 16, 64)));
  if (lg > 5) v = pk_max_u16(v, static_cast<uint32_t>(__shfl_xor(static_cast<int>(v), 32, 64)));
  return v;
}

// One round of the merge across lanes: `a` (descending) against the list of lane ^ X.
template <int KT, int X>
__device__ __forceinline__ void cross_merge(uint32_t (&a)[KT], uint32_t& dropped) {
  uint32_t b[KT];
#pragma unroll
  for (int i = 0; i < KT; ++i) b[i] = quad_xor<X>(a[KT - 1 - i]);
#pragma unroll
  for (int i = 0; i < KT; ++i) {
    dropped = umax(dropped, umin(a[i], b[i]));
    a[i] = umax(a[i], b[i]);
  }
}

// bits 0, 2, 4, 6 of b -> four bytes of all-ones / all-zeros
__device__ __forceinline__ uint32_t spread_even_bits_to_bytes(uint32_t b) {
  const uint32_t t = (b & 1u) | (b & 4u) << 6 | (b & 16u) << 12 | (b & 64u) << 18;
  return (t << 8) - t;
}

template <int B, int KT>
constexpr int lanes_per_bank() { return B / KT >= 4 ? 4 : 2; }

// SHARED: a workgroup is one wave of 64 >> lg_span rows; otherwise it is one row.
template <int B, int KT, bool TIED, bool SHARED>
__global__ __launch_bounds__(SHARED ? 64 : kThreads) void encode_few_kernel(FewEncArgs a) {
  constexpr int LPB = lanes_per_bank<B, KT>(), N = B / LPB;  // channels per lane
  static_assert(N >= KT && N % 8 == 0, "a lane's channels hold the k largest, and whole groups of eight");
  const int tid = threadIdx.x, lane = tid & 63;
  const int at = SHARED ? tid & ((1 << a.lg_span) - 1) : tid;  // lane inside the row
  const int g = at / LPB, q = at % LPB;
  const int64_t row = SHARED ? (static_cast<int64_t>(blockIdx.x) << (6 - a.lg_span)) + (tid >> a.lg_span) : blockIdx.x;
  const bool active = g < a.G && (!SHARED || row < a.M);
  const int c0 = q * N;  // first channel of this lane inside the bank

  uint32_t xr[N / 2];  // bf16 pairs
  {
    const uint4* src = reinterpret_cast<const uint4*>(a.x + (SHARED ? min(row, static_cast<int64_t>(a.M - 1)) : row) * a.ldx +
                                                      static_cast<int64_t>(g < a.G ? g : a.G - 1) * B + c0);
#pragma unroll
    for (int i = 0; i < N / 8; ++i) {
      const uint4 v = src[i];
      xr[4 * i] = v.x;
      xr[4 * i + 1] = v.y;
      xr[4 * i + 2] = v.z;
      xr[4 * i + 3] = v.w;
    }
  }
  // ---- selection: the lane's k largest, then the bank's ----
  uint32_t top[KT], dropped = 0;
  {
    uint32_t key[N];
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {  // (255 - channel) << 1, see make_key; c0 is not a constant
      key[2 * i] = (__builtin_amdgcn_alignbit(xr[i], xr[i], 15) & 0xFFFE0001u) | static_cast<uint32_t>((255 - 2 * i - c0) << 1);
      key[2 * i + 1] = (__builtin_amdgcn_alignbit(xr[i], xr[i], 31) & 0xFFFE0001u) | static_cast<uint32_t>((254 - 2 * i - c0) << 1);
    }
#pragma unroll
    for (int g0 = 0; g0 < N; g0 += KT) sort_desc<KT>(key + g0);
#pragma unroll
    for (int width = KT; width < N; width <<= 1) {
#pragma unroll
      for (int base = 0; base < N; base += 2 * width) {
#pragma unroll
        for (int i = 0; i < KT; ++i) {
          const uint32_t ai = key[base + i], bj = key[base + width + KT - 1 - i];
          dropped = umax(dropped, umin(ai, bj));
          key[base + i] = umax(ai, bj);
        }
        bitonic_merge_desc<KT>(key + base);
      }
    }
#pragma unroll
    for (int i = 0; i < KT; ++i) top[i] = key[i];
  }
  cross_merge<KT, 1>(top, dropped);
  if constexpr (LPB == 4) {
    bitonic_merge_desc<KT>(top);
    cross_merge<KT, 2>(top, dropped);
  }
  uint32_t tmax = top[0];
#pragma unroll
  for (int i = 1; i < KT; ++i) tmax = umax(tmax, top[i]);

  // ---- the row's maxima, per-token scales ----
  uint32_t mx = span_pk_max(active ? (key_magnitude(tmax) << 16) | key_magnitude(dropped) : 0u, SHARED ? a.lg_span : 6);
  if constexpr (!SHARED) {
    __shared__ uint32_t part[kThreads / 64];
    if (lane == 0) part[tid >> 6] = mx;
    __syncthreads();
    for (int w = 0; w < static_cast<int>(blockDim.x) / 64; ++w) mx = pk_max_u16(mx, part[w]);
  }
  if (!active) return;
  const uint32_t mag_hi = mx >> 16, mag_lo = mx & 0xFFFFu;
  const float amax_hi = __uint_as_float(mag_hi << 16), amax_lo = __uint_as_float(mag_lo << 16);
  float inv_hi, inv_lo, sc_hi, sc_lo;
  if constexpr (TIED) {  // as in the streaming encoder
    const float A = fmaxf(amax_hi, __fmul_rn(amax_lo, 127.0f / 112.0f));
    const bool nz = A != 0.0f;
    inv_hi = nz ? 127.0f / A : 0.0f;
    sc_hi = nz ? A / 127.0f : 1.0f;
    inv_lo = __fmul_rn(inv_hi, 0.0625f);
    sc_lo = __fmul_rn(sc_hi, 16.0f);
  } else {
    inv_hi = mag_hi ? a.q_hi / amax_hi : 0.0f;
    inv_lo = mag_lo ? a.q_lo / amax_lo : 0.0f;
    sc_hi = mag_hi ? amax_hi / a.q_hi : 1.0f;
    sc_lo = mag_lo ? amax_lo / a.q_lo : 1.0f;
  }
  if (at == 0) {
    a.s_hi[row] = sc_hi;
    a.s_lo[row] = sc_lo;
  }

  // ---- mask, and the high codes in channel order (every lane of the bank has the set; the first one stores) ----
  uint32_t mw[B / 32];
#pragma unroll
  for (int w = 0; w < B / 32; ++w) mw[w] = 0;
#pragma unroll
  for (int t = 0; t < KT; ++t) {
    const uint32_t ch = key_channel(top[t]);
#pragma unroll
    for (int w = 0; w < B / 32; ++w) mw[w] |= ((ch >> 5) == static_cast<uint32_t>(w)) ? (1u << (ch & 31u)) : 0u;
  }
  if (q == 0) {
    uint32_t ent[KT];  // channel << 8 | code byte
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      const float r = __fadd_rn(__fmul_rn(key_value(top[t]), inv_hi), kRoundMagic);
      ent[t] = (key_channel(top[t]) << 8) | (__float_as_uint(r) & 0xFFu);
    }
    sort_desc<KT>(ent);  // descending channel; read back reversed
    uint32_t hv[(KT + 3) / 4];
#pragma unroll
    for (int i = 0; i < (KT + 3) / 4; ++i) hv[i] = 0;
#pragma unroll
    for (int t = 0; t < KT; ++t) hv[t / 4] |= (ent[KT - 1 - t] & 0xFFu) << (8 * (t % 4));
    store_bytes<KT>(a.hi_val + (row * a.G + g) * KT, hv);
    uint32_t* mdst = a.mask + row * (a.K / 32) + static_cast<int64_t>(g) * (B / 32);
#pragma unroll
    for (int w = 0; w < B / 32; ++w) mdst[w] = mw[w];
  }

  // ---- the lane's own channels: low codes, and the matrix-core-ready image (inside every group of 8 channels the even
  // ones first, then the odd ones) ----
  uint32_t dl[N / 8], im[N / 4];
#pragma unroll
  for (int j = 0; j < N / 8; ++j) {
    const int c = c0 + 8 * j;  // its 8 mask bits: word c / 32, which depends on the lane
    uint32_t word = mw[0];
#pragma unroll
    for (int w = 1; w < B / 32; ++w) word = (c >> 5) == w ? mw[w] : word;
    const uint32_t m8 = (word >> (c & 31)) & 0xFFu;
    dl[j] = quant_lo8(xr + 4 * j, inv_lo) & ~spread_bits_to_nibbles(m8);
    uint32_t ev = 0, od = 0;  // codes at the high scale, kept where the channel is high
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t w = xr[4 * j + e];
      ev = __builtin_amdgcn_alignbit(__float_as_uint(__fadd_rn(__fmul_rn(__uint_as_float(w << 16), inv_hi), kRoundMagic)), ev, 8);
      od = __builtin_amdgcn_alignbit(__float_as_uint(__fadd_rn(__fmul_rn(__uint_as_float(w & 0xFFFF0000u), inv_hi), kRoundMagic)), od, 8);
    }
    im[2 * j] = ev & spread_even_bits_to_bytes(m8);
    im[2 * j + 1] = od & spread_even_bits_to_bytes(m8 >> 1);
    if constexpr (TIED) {  // 16 x the low codes elsewhere
      im[2 * j] |= (dl[j] << 4) & 0xF0F0F0F0u;
      im[2 * j + 1] |= dl[j] & 0xF0F0F0F0u;
    }
  }
  store_bytes<N / 2>(reinterpret_cast<int8_t*>(a.d_lo) + row * (a.K / 2) + static_cast<int64_t>(g) * (B / 2) + c0 / 2, dl);
  if (a.image) store_bytes<N>(a.image + row * a.K + static_cast<int64_t>(g) * B + c0, im);
}

// Threads of a row of `lanes` lanes.
int span_of(int lanes) {
  if (lanes > 32) return (lanes + 63) / 64 * 64;
  int span = 2;
  while (span < lanes) span *= 2;
  return span;
}

template <int B, int KT>
int launch_few_enc(const sq_params& p, FewEncArgs a, bool tied, hipStream_t st) {
  const int span = span_of(a.G * lanes_per_bank<B, KT>());
  if (span < 64) {
    const int rows = 64 / span;
    const dim3 grid((p.M + rows - 1) / rows);
    a.lg_span = __builtin_ctz(span);
    if (tied) hipLaunchKernelGGL((encode_few_kernel<B, KT, true, true>), grid, dim3(64), 0, st, a);
    else hipLaunchKernelGGL((encode_few_kernel<B, KT, false, true>), grid, dim3(64), 0, st, a);
  } else {
    a.lg_span = 6;
    if (tied) hipLaunchKernelGGL((encode_few_kernel<B, KT, true, false>), dim3(p.M), dim3(span), 0, st, a);
    else hipLaunchKernelGGL((encode_few_kernel<B, KT, false, false>), dim3(p.M), dim3(span), 0, st, a);
  }
  return hipGetLastError() == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}

}  // namespace

// Which calls.  Splitting a bank in four costs about 1.7 times its instructions in all, so up to eight waves per compute unit
// (workgroups per unit times waves each): 8 waves [256,8192] 4.7 against 6.5 us, 10 waves [300,5120] 6.0 against 5.7 us,
// 22 waves [333,11008] 9.3 against 8.3 us.  Split in two the chain is hardly shorter, so only while no SIMD has two waves:
// k = 32 of b = 64 [1024,2048] 6.8 against 9.2 us, but [2048,2048] 10.3 against 9.3 us; and several workgroups of more than
// one wave do not spread evenly over the SIMDs ([512,4096] 9.6 against 8.7 us).  Rows of b = 32 that leave lanes of a shared
// wave idle lose from the fifth wave on ([2202,192] 3.8 against 3.7 us).
bool encode_few_supports(const sq_params& p) {
  const int lpb = p.bank / p.topk >= 4 ? 4 : 2, lanes = p.K / p.bank * lpb, cus = device_compute_units();
  if (lanes > kThreads) return false;
  const int span = span_of(lanes), waves = (span + 63) / 64, rows = span < 64 ? 64 / span : 1;
  const int64_t groups = (p.M + rows - 1) / rows, per_cu = (groups + cus - 1) / cus;  // workgroups in all, and per compute unit
  if (lpb == 2) return per_cu * waves <= 4 && (per_cu == 1 || waves == 1);
  return per_cu * waves <= (p.bank == 32 && span < 64 && lanes < span ? 4 : 8);
}

int launch_encode_few(const sq_params& p, const uint16_t* x, int64_t ldx, const sq_act& out, bool tied, hipStream_t st) {
  FewEncArgs a;
  a.x = x;
  a.ldx = ldx;
  a.M = p.M;
  a.K = p.K;
  a.G = p.K / p.bank;
  a.d_lo = out.d_lo;
  a.hi_val = out.hi_val;
  a.mask = out.mask;
  a.s_lo = out.scale_lo;
  a.s_hi = out.scale_hi;
  a.image = out.hi_dense;
  a.q_hi = tied ? 127.0f : code_max(p.h_high, 8);
  a.q_lo = tied ? 7.0f : code_max(p.h_low, 4);
#define SQ_CASE(B, KT) \
  if (p.bank == B && p.topk == KT) return launch_few_enc<B, KT>(p, a, tied, st);
  SQ_CASE(32, 2) SQ_CASE(32, 4) SQ_CASE(32, 8) SQ_CASE(32, 16)
  SQ_CASE(64, 4) SQ_CASE(64, 8) SQ_CASE(64, 16) SQ_CASE(64, 32)
  SQ_CASE(128, 8) SQ_CASE(128, 16) SQ_CASE(128, 32)
#undef SQ_CASE
  return SQ_ERR_UNSUPPORTED;
}

}  // namespace sq
