// sq_gemm for few tokens (M <= 64): the layer is a stream over the INT4 weights, and the work of one output
// channel is so small that channels alone do not fill the chip (a 4096-channel layer is 64 workgroups of 64).
// Every wave of a workgroup therefore takes a share of K (K steps wave, wave + NW, ...) of ALL the workgroup's
// outputs, and the integer partial sums -- exact in any order -- meet in LDS at the end.
//
// A wave owns a private ring of LDS stages, filled by its own LDS-direct loads and read by nobody else, so the
// K loop has no barrier at all: it waits on its own counter, reads a stage, refills it and multiplies.  (The
// kernel it replaces met at a workgroup barrier on every 128 channels and spent most of a step on that chain.)
// Matrix instruction: v_mfma_i32_16x16x64_i8, weights as the row operand, so that a lane ends up with four
// consecutive output channels of one token.
//
// A 128-channel step of a packed row is four 16-byte chunks; lane group q (lane / 16) holds chunk q, i.e. the
// channels 32 q ... 32 q + 31, and widens half s of it for matrix instruction s (see sq_gemm.hip for the widening
// and for the byte order of the INT8 operands, which is the same here).
#include <type_traits>

#include "sq_device.h"
#include "sq_gemm_common.h"

namespace sq {
namespace {

using namespace gemm;

constexpr int kLds = 160 * 1024;

// MODE 0: low + zero-padded high in one loop (dynamic); 1: the low steps, then the compact high steps (static);
// 2: one INT8 operand (tied scales, plain W4A8).  MT: tokens staged (8, 16, 32, 48, 64); CT: 16-channel tiles.
template <int MODE_, int MT_, int CT_>
struct FewCfg {
  static constexpr int MODE = MODE_, MT = MT_, CT = CT_;
  static constexpr int RT = MT < 16 ? 1 : MT / 16;       // 16-token tiles
  static constexpr int BN = 16 * CT;
  static constexpr int A_OFF = CT * 1024;                // stage: weights [BN][64 B], then the activation tiles
  static constexpr int A_HI = A_OFF + (MODE == 0 ? MT * 64 : 0);
  static constexpr int STAGE = A_HI + MT * 128;          // MODE 1: a low step uses half of the activation area
  static constexpr int N_LO = MT < 16 ? 1 : MT / 16;     // copies of a step: low codes, INT8 codes
  static constexpr int N_HI = MT / 8;
  static constexpr int NL = CT + (MODE == 0 ? N_LO + N_HI : (MODE == 1 ? N_LO : N_HI));  // (MODE 1: of a low step, the smaller number)
  // waves: as many as leave room for two stages each, and for the accumulators of more than 16 tokens
  static constexpr int NW = MT > 16 ? 4 : (16 * STAGE <= kLds ? 8 : 6);
  static constexpr int DMAX = kLds / (NW * STAGE);
  static constexpr int D = DMAX > 4 ? 4 : DMAX;          // stages of a wave's ring
  static constexpr int PARTS = MODE == 2 ? 1 : 2;
  static constexpr int TILES = RT * CT;
  static constexpr int TILE_BYTES = NW * PARTS * 1024;   // one 16 x 16 tile's partial sums of all waves
  static constexpr int TPP = kLds / TILE_BYTES < TILES ? kLds / TILE_BYTES : TILES;  // tiles reduced per pass
  static constexpr int RING = NW * D * STAGE;
  static constexpr int LDS_BYTES = RING > TPP * TILE_BYTES ? RING : TPP * TILE_BYTES;
  static_assert(D >= 2 && (D - 1) * NL < 64 && LDS_BYTES <= kLds, "ring");
};

template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void wait_lgkm0() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((15) | (7 << 4) | (0 << 8) | (3 << 14));
  asm volatile("" ::: "memory");
}

// The copies of up to D - 1 later steps may be in flight.
template <int D, int NL>
__device__ __forceinline__ void wait_step(int later) {
  if constexpr (D > 3) {
    if (later >= 3) { wait_vm<3 * NL>(); return; }
  }
  if constexpr (D > 2) {
    if (later >= 2) { wait_vm<2 * NL>(); return; }
  }
  if (later >= 1) wait_vm<NL>();
  else wait_vm<0>();
}

// Sources of one operand pair (weights and activations) of the K loop.
struct FewSrc {
  const char* w;     // weights of the workgroup's first channel
  const char* a_lo;  // packed codes, or null
  const char* a_hi;  // INT8 codes, or null
  int64_t ldw, lda_lo, lda_hi;
  int kext;          // channels
};

template <typename C, bool LO, bool HI>
__device__ __forceinline__ void few_issue(const GemmArgs& g, const FewSrc& s, char* stage, int step, int n0, int lane) {
  const int k0 = step * 128;
  const bool tail = k0 + 128 > s.kext;  // uniform
  const char* zero = reinterpret_cast<const char*>(kZeroChunk);
  const int c4 = ((lane & 3) ^ (lane >> 4)) & 3;  // chunk of a 64-byte row that this lane's 16 bytes hold (off4)
  const bool ok4 = !tail || k0 + c4 * 32 < s.kext;
  const int nmax = g.N - 1 - n0;
#pragma unroll
  for (int j = 0; j < C::CT; ++j) {
    const int row = min(16 * j + (lane >> 2), nmax);
    const char* src = s.w + (k0 >> 1) + (static_cast<int64_t>(row) * s.ldw + c4 * 16);
    if (tail) src = ok4 ? src : zero;
    __builtin_amdgcn_global_load_lds(src, (lds_ptr_t)(stage + j * 1024), 16, 0, 0);
  }
  if constexpr (LO) {
#pragma unroll
    for (int i = 0; i < C::N_LO; ++i) {
      const int row = min(16 * i + (lane >> 2), g.M - 1);
      const char* src = s.a_lo + (k0 >> 1) + (static_cast<int64_t>(row) * s.lda_lo + c4 * 16);
      if (tail) src = ok4 ? src : zero;
      if (C::MT >= 16 || lane < 32)  // 8 tokens: half a wave's worth
        __builtin_amdgcn_global_load_lds(src, (lds_ptr_t)(stage + C::A_OFF + i * 1024), 16, 0, 0);
    }
  }
  if constexpr (HI) {
    constexpr int off = C::MODE == 1 ? C::A_OFF : C::A_HI;
#pragma unroll
    for (int i = 0; i < C::N_HI; ++i) {
      const int r0 = 8 * i + (lane >> 3);
      const int c8 = ((lane & 7) ^ (r0 >> 1)) & 7;
      const char* src = s.a_hi + k0 + (static_cast<int64_t>(min(r0, g.M - 1)) * s.lda_hi + c8 * 16);
      if (tail) src = k0 + c8 * 16 < s.kext ? src : zero;
      __builtin_amdgcn_global_load_lds(src, (lds_ptr_t)(stage + off + i * 1024), 16, 0, 0);
    }
  }
}

template <typename C>
struct FewAcc {
  v4i lo[C::RT][C::CT], hi[C::RT][C::CT];
};

template <typename C>
struct FewFrags {
  v4u w[C::CT];
  v4u lo[C::RT];
  v4i hi[C::RT][2];
};

template <typename C, bool LO, bool HI>
__device__ __forceinline__ void few_read(FewFrags<C>& f, const char* stage, int lane) {
  const int r = lane & 15, q = lane >> 4;
  const int ra = C::MT < 16 ? (r & (C::MT - 1)) : r;  // 8 tokens: the other eight columns repeat them (never stored)
#pragma unroll
  for (int j = 0; j < C::CT; ++j) f.w[j] = *reinterpret_cast<const v4u*>(stage + off4(16 * j + r, q));
#pragma unroll
  for (int i = 0; i < C::RT; ++i) {
    if (LO) f.lo[i] = *reinterpret_cast<const v4u*>(stage + C::A_OFF + off4(16 * i + ra, q));
    if (HI) {
      constexpr int off = C::MODE == 1 ? C::A_OFF : C::A_HI;
      f.hi[i][0] = *reinterpret_cast<const v4i*>(stage + off + off8(16 * i + ra, 2 * q));
      f.hi[i][1] = *reinterpret_cast<const v4i*>(stage + off + off8(16 * i + ra, 2 * q + 1));
    }
  }
}

template <typename C, bool LO, bool HI>
__device__ __forceinline__ void few_mma(FewAcc<C>& a, const FewFrags<C>& f) {
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    v4i alo[C::RT];
    if (LO) {
#pragma unroll
      for (int i = 0; i < C::RT; ++i) alo[i] = widen(f.lo[i], s);
    }
#pragma unroll
    for (int j = 0; j < C::CT; ++j) {
      const v4i bw = widen(f.w[j], s);
#pragma unroll
      for (int i = 0; i < C::RT; ++i) {
        if (LO) a.lo[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bw, alo[i], a.lo[i][j], 0, 0, 0);
        if (HI) a.hi[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bw, f.hi[i][s], a.hi[i][j], 0, 0, 0);
      }
    }
  }
}

template <typename C>
__global__ __launch_bounds__(64 * C::NW) void gemm_few_kernel(GemmArgs g) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  constexpr int MODE = C::MODE, D = C::D, NW = C::NW;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n0 = blockIdx.x * C::BN;
  const int r = lane & 15, q = lane >> 4;

  FewSrc s1, s2;  // s2: the compact high steps of MODE 1
  if constexpr (MODE == 0) {
    s1 = {reinterpret_cast<const char*>(g.wq) + static_cast<int64_t>(n0) * (g.K / 2), reinterpret_cast<const char*>(g.a_lo),
          reinterpret_cast<const char*>(g.a_hi_dense), g.K / 2, g.K / 2, g.K, g.K};
    s2 = s1;
  } else {
    s1 = {reinterpret_cast<const char*>(g.w_lo) + static_cast<int64_t>(n0) * (g.K_lo / 2), reinterpret_cast<const char*>(g.a_lo),
          nullptr, g.K_lo / 2, g.K_lo / 2, 0, g.K_lo};
    s2 = {reinterpret_cast<const char*>(g.w_hi) + static_cast<int64_t>(n0) * (g.K_hi / 2), nullptr,
          reinterpret_cast<const char*>(g.a_hi_compact), g.K_hi / 2, 0, g.lda_hi_compact, g.K_hi};
  }
  const int steps1 = MODE == 2 ? 0 : (s1.kext + 127) / 128;
  const int steps = steps1 + (MODE == 0 ? 0 : (s2.kext + 127) / 128);
  const int mine = wave < steps ? (steps - wave + NW - 1) / NW : 0;  // steps of this wave
  char* ring = lds + wave * (D * C::STAGE);

  // The workgroups of an XCD start at different places of K (the steps wrap around): in step with each other they
  // would ask for the same few hundred bytes of every weight row at a time, and with rows 4 KB apart those lie in a
  // fraction of the memory channels ([8,8192] x [28672,8192]: 27.2 us in step, 24.5 us turned).
  const int turn = (blockIdx.x >> 3) * NW;
  const int turn1 = MODE == 2 ? 0 : turn % steps1, turn2 = MODE == 0 ? 0 : turn % (steps - steps1);
  auto issue = [&](char* stage, int step) {
    if (MODE == 0 || (MODE == 1 && step < steps1)) {
      step += turn1;
      few_issue<C, true, MODE == 0>(g, s1, stage, step >= steps1 ? step - steps1 : step, n0, lane);
    } else if constexpr (MODE != 0) {
      step += turn2;
      few_issue<C, false, true>(g, s2, stage, (step >= steps ? step - (steps - steps1) : step) - steps1, n0, lane);
    }
  };
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (d < mine) issue(ring + d * C::STAGE, wave + d * NW);

  FewAcc<C> acc;
#pragma unroll
  for (int i = 0; i < C::RT; ++i)
#pragma unroll
    for (int j = 0; j < C::CT; ++j) {
      acc.lo[i][j] = v4i{0, 0, 0, 0};
      acc.hi[i][j] = v4i{0, 0, 0, 0};
    }

  int st = 0, i = 0;
  auto body = [&](auto lo, auto hi) {
    constexpr bool LO = decltype(lo)::value, HI = decltype(hi)::value;
    char* stage = ring + st * C::STAGE;
    st = st == D - 1 ? 0 : st + 1;
    // (MODE 1 counts every later step as a low one, which has fewer copies: the wait is then for a little more)
    wait_step<D, C::NL>(mine - 1 - i);
    FewFrags<C> f;
    few_read<C, LO, HI>(f, stage, lane);
    wait_lgkm0();  // the stage is in registers: refill it
    if (i + D < mine) issue(stage, wave + (i + D) * NW);
    few_mma<C, LO, HI>(acc, f);
    ++i;
  };
  using T = std::true_type;
  using F = std::false_type;
  if constexpr (MODE == 0) {
    while (i < mine) body(T{}, T{});
  } else {
    if constexpr (MODE == 1)
      while (i < mine && wave + i * NW < steps1) body(T{}, F{});
    while (i < mine) body(F{}, T{});
  }

  // ---- the waves' partial sums meet in LDS, TPP tiles at a time; wave t % NW adds up tile t and stores it ----
#pragma unroll
  for (int p0 = 0; p0 < C::TILES; p0 += C::TPP) {
    __syncthreads();  // the rings (first pass) or the previous pass have been read
#pragma unroll
    for (int t = p0; t < p0 + C::TPP && t < C::TILES; ++t) {
      char* dst = lds + (t - p0) * C::TILE_BYTES + wave * (C::PARTS * 1024) + lane * 16;
      if constexpr (MODE != 2) {
        *reinterpret_cast<v4i*>(dst) = acc.lo[t / C::CT][t % C::CT];
        *reinterpret_cast<v4i*>(dst + 1024) = acc.hi[t / C::CT][t % C::CT];
      } else {
        *reinterpret_cast<v4i*>(dst) = acc.hi[t / C::CT][t % C::CT];
      }
    }
    __syncthreads();
    const int tn = min(C::TPP, C::TILES - p0);
    for (int t = wave; t < tn; t += NW) {
      const int rt = (p0 + t) / C::CT, ct = (p0 + t) % C::CT;
      const char* src = lds + t * C::TILE_BYTES + lane * 16;
      v4i lo = {0, 0, 0, 0}, hi = {0, 0, 0, 0};
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        if constexpr (MODE != 2) {
          lo += *reinterpret_cast<const v4i*>(src + w * 2048);
          hi += *reinterpret_cast<const v4i*>(src + w * 2048 + 1024);
        } else {
          hi += *reinterpret_cast<const v4i*>(src + w * 1024);
        }
      }
      const int m = rt * 16 + r, n = n0 + ct * 16 + 4 * q;
      if ((C::MT < 16 && r >= C::MT) || m >= g.M || n >= g.N) continue;
      const float slo = MODE != 2 ? g.s_lo[m] : 0.0f, shi = g.s_hi[m];
      float y[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float t2 = MODE != 2 ? __fmul_rn(static_cast<float>(lo[e] >> 8), slo) : 0.0f;
        t2 = __fmaf_rn(static_cast<float>(hi[e] >> 4), shi, t2);
        y[e] = __fmul_rn(t2, g.s_w[min(n + e, g.N - 1)]);
      }
      const int64_t o = static_cast<int64_t>(m) * g.ldy + n;
      const bool vec = n + 4 <= g.N && (g.ldy & 3) == 0;
      if (g.out_bf16) {
        uint16_t* yo = reinterpret_cast<uint16_t*>(g.y) + o;
        if (vec) {
          *reinterpret_cast<v2u*>(yo) = v2u{bf16_rne(y[0]) | static_cast<unsigned>(bf16_rne(y[1])) << 16,
                                            bf16_rne(y[2]) | static_cast<unsigned>(bf16_rne(y[3])) << 16};
        } else {
          for (int e = 0; e < 4 && n + e < g.N; ++e) yo[e] = bf16_rne(y[e]);
        }
      } else {
        float* yo = reinterpret_cast<float*>(g.y) + o;
        if (vec) *reinterpret_cast<f32x4*>(yo) = f32x4{y[0], y[1], y[2], y[3]};
        else
          for (int e = 0; e < 4 && n + e < g.N; ++e) yo[e] = y[e];
      }
      for (int e = 0; e < 4 && n + e < g.N; ++e) {  // test hook: the exact accumulators
        if (g.acc_lo_dbg) g.acc_lo_dbg[static_cast<int64_t>(m) * g.N + n + e] = lo[e] >> 8;
        if (g.acc_hi_dbg) g.acc_hi_dbg[static_cast<int64_t>(m) * g.N + n + e] = hi[e] >> 4;
      }
    }
  }
}

template <typename C>
int launch_few_t(const GemmArgs& g, hipStream_t st) {
  hipLaunchKernelGGL((gemm_few_kernel<C>), dim3((g.N + C::BN - 1) / C::BN), dim3(64 * C::NW), C::LDS_BYTES, st, g);
  return hipGetLastError() == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}

template <typename C>
hipError_t raise_few() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_few_kernel<C>), hipFuncAttributeMaxDynamicSharedMemorySize,
                             C::LDS_BYTES);
}

#define SQ_FEW_CT(X, MODE, CT) X(MODE, 8, CT) X(MODE, 16, CT) X(MODE, 32, CT)
#define SQ_FEW_MODE(X, MODE)                                                                                       \
  SQ_FEW_CT(X, MODE, 1) SQ_FEW_CT(X, MODE, 2) SQ_FEW_CT(X, MODE, 3) SQ_FEW_CT(X, MODE, 4) SQ_FEW_CT(X, MODE, 5)    \
  SQ_FEW_CT(X, MODE, 6) SQ_FEW_CT(X, MODE, 7) SQ_FEW_CT(X, MODE, 8)                                                \
  X(MODE, 48, 1) X(MODE, 48, 2) X(MODE, 64, 1) X(MODE, 64, 2)
#define SQ_FEW_CASES(X) SQ_FEW_MODE(X, 0) SQ_FEW_MODE(X, 1) SQ_FEW_MODE(X, 2)

int launch_few_shape(const GemmArgs& g, int mode, int mt, int ct, hipStream_t st) {
#define X(MODE, MT, CT) \
  if (mode == MODE && mt == MT && ct == CT) return launch_few_t<FewCfg<MODE, MT, CT>>(g, st);
  SQ_FEW_CASES(X)
#undef X
  return SQ_ERR_UNSUPPORTED;
}

}  // namespace

// 33 ... 64 tokens: worth it only where the 64-channel tiles would cover at most half of the chip.
bool gemm_few_supports(int M, int N) { return M <= 32 || (M <= 64 && N <= 8192); }

int init_gemm_few_kernels() {
  hipError_t e = hipSuccess;
#define X(MODE, MT, CT) \
  if (e == hipSuccess) e = raise_few<FewCfg<MODE, MT, CT>>();
  SQ_FEW_CASES(X)
#undef X
  return e == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}

void gemm_few_shape(int M, int N, int* rows, int* ct) {
  const int mt = M <= 8 ? 8 : (M + 15) / 16 * 16;
  *rows = mt;  // 8, 16, 32, 48 or 64
  // Channels per workgroup: one workgroup fills a compute unit, so the rounds over the chip count, and each costs
  // the workgroup's channels plus about one tile's worth of activations, start and end.
  int best = 1 << 30;
  for (int c = 1; c <= (mt > 32 ? 2 : 8); ++c) {
    const int groups = (N + 16 * c - 1) / (16 * c);
    const int cost = (groups + 255) / 256 * (c + 1);
    if (cost <= best) {
      best = cost;
      *ct = c;
    }
  }
}

int launch_gemm_few(const GemmArgs& g, int mode, hipStream_t st) {
  int rows, ct;
  gemm_few_shape(g.M, g.N, &rows, &ct);
  return launch_few_shape(g, mode, rows, ct, st);
}

}  // namespace sq
