// The SQ-format at its equivalent bit width (Section 4.1: y = (1-s)*h_high + s*h_low bits per element):
// conversion between the compute containers of an sq_act (INT8 high codes, 4-bit low codes dense over K)
// and the packed stream -- per token row the high codes of the high channels at h_high bits each, then the low
// codes of the low channels only at h_low bits each, ascending channel order, least significant bit first.
//
// Bound by HBM in both directions.  A workgroup converts a few whole rows (consecutive bytes of the stream) through an
// image of them in LDS: the image starts at the stream's own offset inside 16 bytes, so that whatever the length of a row
// the stream is read and written 16 bytes at a time, and bit fields of any width and place are ORed into, or cut out of,
// LDS dwords.  A thread converts 32 channels at a time.  With one thread per byte of the stream, which looked its channel
// up in the mask, [4096,4096] took 110 us to pack and 33 us to unpack, against 8.7 and 11.1 us.  Short calls are launch and
// latency only and pack without the image (pack_by_bytes).
#include "sq_gemm_common.h"

namespace sq {
namespace {

using gemm::v4u;

constexpr int kThreads = 256;  // threads of a workgroup (twice as many for long rows)

struct StoreArgs {
  int M, K, B, kt, hh, hl;
  int K_hi;
  int row_bytes, hi_bytes;
  int rows;             // rows per workgroup
  int64_t mask_stride;  // words between the masks of consecutive rows (0: one mask for all rows)
  const uint32_t* mask;
  uint32_t* mask_out;   // sentinel form, unpack: the mask recovered from the sentinels
  uint8_t* d_lo;
  int8_t* hi_val;
  uint8_t* packed;
};

// What every thread of a workgroup knows about its rows.  Bit and byte positions count from the start of the image.
struct Span {
  int64_t m0;
  int rows, phase, end;  // image bytes [phase, end) are the rows
  uint8_t* stream;       // the rows in memory
  __device__ __forceinline__ Span(const StoreArgs& a) {
    m0 = static_cast<int64_t>(blockIdx.x) * a.rows;
    rows = static_cast<int>(min(static_cast<int64_t>(a.rows), a.M - m0));
    stream = a.packed + m0 * a.row_bytes;
    phase = static_cast<int>(reinterpret_cast<uintptr_t>(stream) & 15);
    end = phase + rows * a.row_bytes;
  }
};

// ORs the low n bits of x (n <= 32; the others are zero) into the image at `bit`, as far as they lie before `limit`.
__device__ __forceinline__ void or_bits(uint32_t* img, int bit, uint32_t x, int n, int limit) {
  if (bit + n > limit) x = bit < limit ? x & ((1u << (limit - bit)) - 1u) : 0u;
  const uint64_t v = static_cast<uint64_t>(x) << (bit & 31);
  if (static_cast<uint32_t>(v)) atomicOr(img + (bit >> 5), static_cast<uint32_t>(v));
  if (v >> 32) atomicOr(img + (bit >> 5) + 1, static_cast<uint32_t>(v >> 32));
}
// 32 bits of the image from `bit` on; those from `limit` on read as zero.
__device__ __forceinline__ uint32_t bits32(const uint32_t* img, int bit, int limit) {
  if (bit >= limit) return 0;
  const uint64_t two = img[bit >> 5] | static_cast<uint64_t>(img[(bit >> 5) + 1]) << 32;
  const uint32_t v = static_cast<uint32_t>(two >> (bit & 31));
  return bit + 32 > limit ? v & ((1u << (limit - bit)) - 1u) : v;
}

// Low channels of word w's bank before the word (an explicit mask row).
__device__ __forceinline__ int lows_before(const uint32_t* mrow, int w, int wpb) {
  const int w0 = w / wpb * wpb;
  int n = (w - w0) * 32;
  for (int i = w0; i < w; ++i) n -= __popc(mrow[i]);
  return n;
}

template <int NT, bool SENTINEL>
__global__ __launch_bounds__(NT) void pack_storage_kernel(StoreArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint32_t img[];
  const Span s(a);
  const int tid = threadIdx.x;
  for (int i = tid; i < (s.end + 15) / 16; i += NT) reinterpret_cast<v4u*>(img)[i] = v4u{0u, 0u, 0u, 0u};
  __syncthreads();
  const int hpr = a.K_hi / 4;  // dwords of high codes per row
  const uint32_t* hv = reinterpret_cast<const uint32_t*>(a.hi_val) + s.m0 * hpr;
  for (int i = tid; i < s.rows * hpr; i += NT) {
    const int r = i / hpr, bit0 = 8 * (s.phase + r * a.row_bytes);
    const uint32_t v = hv[i];
    if (a.hh == 8) {
      or_bits(img, bit0 + 32 * (i - r * hpr), v, 32, 8 * s.end);
    } else {
      const uint32_t n = v & 0x0F0F0F0Fu, p = n | (n >> 4);
      or_bits(img, bit0 + 16 * (i - r * hpr), (p & 0xFFu) | ((p >> 8) & 0xFF00u), 16, 8 * s.end);
    }
  }
  const int wpr = a.K / 32, wpb = a.B / 32, nlo = a.B - a.kt;
  const uint32_t cmask = (1u << a.hl) - 1u, v_mask = 1u << (a.hl - 1);
  for (int i = tid; i < s.rows * wpr; i += NT) {
    const int r = i / wpr, w = i - r * wpr;
    const uint32_t* mrow = a.mask + (s.m0 + r) * a.mask_stride;
    const uint32_t word = mrow[w];
    const v4u d = *reinterpret_cast<const v4u*>(a.d_lo + (s.m0 + r) * (a.K / 2) + static_cast<int64_t>(w) * 16);
    const int limit = 8 * (s.phase + (r + 1) * a.row_bytes);
    int bit = 8 * (s.phase + r * a.row_bytes + a.hi_bytes), left = 0;
    if constexpr (SENTINEL) {
      bit += 32 * w * a.hl;
    } else {
      const int before = min(lows_before(mrow, w, wpb), nlo);
      bit += (w / wpb * nlo + before) * a.hl;
      left = nlo - before;  // a bank has no more low codes than that, whatever the mask holds
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t x = 0;
      int n = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool hi = (word >> (8 * q + e)) & 1u;
        const uint32_t code = (d[q] >> (4 * e)) & cmask;
        if constexpr (SENTINEL) {  // every channel has a code; the high ones carry the unused most negative one
          x |= (hi ? v_mask : code) << (a.hl * e);
        } else if (!hi && left > 0) {
          x |= code << n;
          n += a.hl;
          --left;
        }
      }
      if constexpr (SENTINEL) n = 8 * a.hl;
      or_bits(img, bit, x, n, limit);
      bit += n;
    }
  }
  __syncthreads();
  // image -> stream: whole 16-byte pieces, single bytes at the two ends
  const char* img8 = reinterpret_cast<const char*>(img);
  const int b0 = (s.phase + 15) / 16 * 16, b1 = max(s.end / 16 * 16, b0);
  uint8_t* at = s.stream - s.phase;
  for (int i = b0 / 16 + tid; i < b1 / 16; i += NT) *reinterpret_cast<v4u*>(at + 16 * i) = reinterpret_cast<const v4u*>(img)[i];
  for (int i = s.phase + tid; i < min(b0, s.end); i += NT) at[i] = static_cast<uint8_t>(img8[i]);
  for (int i = b1 + tid; i < s.end; i += NT) at[i] = static_cast<uint8_t>(img8[i]);
}

// Channel of the r-th low channel of a bank of mask words (r counts from 0; in range for a malformed mask, too).
__device__ __forceinline__ int low_channel(const uint32_t* mbank, int wpb, int r) {
  for (int w = 0; w < wpb; ++w) {
    uint32_t z = ~mbank[w];
    const int c = __popc(z);
    if (r < c) {
      int at = 32 * w;
#pragma unroll
      for (int s = 16; s > 0; s >>= 1) {
        const int n = __popc(z & ((1u << s) - 1u));
        if (r >= n) {
          r -= n;
          z >>= s;
          at += s;
        }
      }
      return at;
    }
    r -= c;
  }
  return 0;
}

// Short calls: a thread makes one byte of the stream by itself.
template <bool SENTINEL>
__global__ __launch_bounds__(kThreads) void pack_bytes_kernel(StoreArgs a) {
  const unsigned idx = blockIdx.x * kThreads + threadIdx.x;
  if (idx >= static_cast<unsigned>(a.M) * a.row_bytes) return;
  const int m = idx / a.row_bytes, b = idx - m * a.row_bytes;
  uint32_t out = 0;
  if (b < a.hi_bytes) {
    const uint8_t* h = reinterpret_cast<const uint8_t*>(a.hi_val) + m * a.K_hi;
    out = a.hh == 8 ? h[b] : (h[2 * b] & 0xFu) | (h[2 * b + 1] & 0xFu) << 4;
  } else {
    const uint32_t* mrow = a.mask + m * a.mask_stride;
    const uint8_t* drow = a.d_lo + m * (a.K / 2);
    const int bit0 = 8 * (b - a.hi_bytes), nlo = a.B - a.kt, codes = SENTINEL ? a.K : a.K - a.K_hi;
    const uint32_t cmask = (1u << a.hl) - 1u;
    for (int t = bit0 / a.hl; t * a.hl < bit0 + 8 && t < codes; ++t) {
      int ch = t;
      bool hi = false;
      if constexpr (SENTINEL) {
        hi = (mrow[t >> 5] >> (t & 31)) & 1u;
      } else {
        const int bank = t / nlo;
        ch = bank * a.B + low_channel(mrow + bank * (a.B / 32), a.B / 32, t - bank * nlo);
      }
      const uint32_t code = hi ? 1u << (a.hl - 1) : (static_cast<uint32_t>(drow[ch >> 1]) >> (4 * (ch & 1))) & cmask;
      const int sh = t * a.hl - bit0;
      out |= sh >= 0 ? code << sh : code >> -sh;
    }
  }
  a.packed[idx] = static_cast<uint8_t>(out);
}

template <int NT, bool SENTINEL>
__global__ __launch_bounds__(NT) void unpack_storage_kernel(StoreArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint32_t img[];
  const Span s(a);
  const int tid = threadIdx.x;
  {  // stream -> image
    char* img8 = reinterpret_cast<char*>(img);
    const int b0 = (s.phase + 15) / 16 * 16, b1 = max(s.end / 16 * 16, b0);
    const uint8_t* at = s.stream - s.phase;
    for (int i = b0 / 16 + tid; i < b1 / 16; i += NT) reinterpret_cast<v4u*>(img)[i] = *reinterpret_cast<const v4u*>(at + 16 * i);
    for (int i = s.phase + tid; i < min(b0, s.end); i += NT) img8[i] = static_cast<char>(at[i]);
    for (int i = b1 + tid; i < s.end; i += NT) img8[i] = static_cast<char>(at[i]);
  }
  __syncthreads();
  const int hpr = a.K_hi / 4;
  uint32_t* hv = reinterpret_cast<uint32_t*>(a.hi_val) + s.m0 * hpr;
  for (int i = tid; i < s.rows * hpr; i += NT) {  // the high section has the order of hi_val
    const int r = i / hpr, bit0 = 8 * (s.phase + r * a.row_bytes);
    if (a.hh == 8) {
      hv[i] = bits32(img, bit0 + 32 * (i - r * hpr), 8 * s.end);
    } else {
      const uint32_t p = bits32(img, bit0 + 16 * (i - r * hpr), 8 * s.end);
      const uint32_t n = (p & 0xFu) | (p & 0xF0u) << 4 | (p & 0xF00u) << 8 | (p & 0xF000u) << 12;
      hv[i] = n | ((n & 0x08080808u) >> 3) * 0xF0u;  // sign-extended inside every byte
    }
  }
  const int wpr = a.K / 32, wpb = a.B / 32, nlo = a.B - a.kt;
  const uint32_t cmask = (1u << a.hl) - 1u, v_mask = 1u << (a.hl - 1);
  for (int i = tid; i < s.rows * wpr; i += NT) {
    const int r = i / wpr, w = i - r * wpr;
    const int limit = 8 * (s.phase + (r + 1) * a.row_bytes);
    int bit = 8 * (s.phase + r * a.row_bytes + a.hi_bytes), left = 0;
    uint32_t word = 0;
    if constexpr (SENTINEL) {
      bit += 32 * w * a.hl;
    } else {
      const uint32_t* mrow = a.mask + (s.m0 + r) * a.mask_stride;
      word = mrow[w];
      const int before = min(lows_before(mrow, w, wpb), nlo);
      bit += (w / wpb * nlo + before) * a.hl;
      left = nlo - before;
    }
    v4u d;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t x = bits32(img, bit, limit), out = 0;
      int n = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t code = x & cmask;
        const uint32_t nib = ((code ^ v_mask) - v_mask) & 0xFu;  // sign-extended to four bits
        if constexpr (SENTINEL) {
          if (code == v_mask) word |= 1u << (8 * q + e);
          else out |= nib << (4 * e);
          x >>= a.hl;
        } else if (!((word >> (8 * q + e)) & 1u) && left > 0) {
          out |= nib << (4 * e);
          x >>= a.hl;
          n += a.hl;
          --left;
        }
      }
      bit += SENTINEL ? 8 * a.hl : n;
      d[q] = out;
    }
    *reinterpret_cast<v4u*>(a.d_lo + (s.m0 + r) * (a.K / 2) + static_cast<int64_t>(w) * 16) = d;
    if constexpr (SENTINEL) a.mask_out[(s.m0 + r) * wpr + w] = word;
  }
}

// Which calls pack byte by byte.  The image costs two barriers and its atomics, 0.5 to 2 us more than a short call takes
// without it, but moves 16 bytes per thread; a byte of the sentinel form needs no search, one of the explicit form looks its
// channel up in the mask words, which costs least where half of them are low, and does not pay for banks of 128 or for more
// than two codes a byte.  Byte by byte against the image: sentinel [8,512] 2.1 and 2.6 us, k = 32 of 64 [32,11008] 3.0 and
// 4.8, [128,4096] 3.5 and 3.5, [512,4096] 8.0 and 3.8; explicit k = 32 of 64 [32,4096] 2.9 and 4.0, [512,2048] 5.6 and 3.9,
// k = 8 of 64 [32,4096] 3.1 and 3.4, [512,1024] 4.5 and 3.4, k = 32 of 128 [32,4096] 4.0 and 3.7.
bool pack_by_bytes(const sq_params& p, int hl, bool sentinel) {
  const int64_t n = static_cast<int64_t>(p.M) * p.K;
  if (sentinel) return n <= (hl == 4 || p.K > 8192 ? 1 << 19 : 1 << 18);
  return hl == 4 && p.bank <= 64 && n <= (2 * p.topk == p.bank ? 1 << 19 : 1 << 17);
}

}  // namespace

int launch_storage(const sq_params& p, const sq_act& act, uint8_t* packed, bool pack, bool sentinel, hipStream_t st) {
  StoreArgs a;
  a.M = p.M;
  a.K = p.K;
  a.B = p.bank;
  a.kt = p.topk;
  a.hh = p.h_high ? p.h_high : 8;
  a.hl = p.h_low ? p.h_low : 4;
  a.K_hi = p.K / p.bank * p.topk;  // a multiple of 4 for every format
  a.hi_bytes = a.K_hi * a.hh / 8;
  a.row_bytes = a.hi_bytes + ((sentinel ? p.K : p.K - a.K_hi) * a.hl + 7) / 8;  // (8/3) may end in half a byte, padded with zeros
  a.mask_out = act.mask;
  a.mask_stride = p.mode == SQ_STATIC ? 0 : p.K / 32;
  a.mask = act.mask;
  a.d_lo = act.d_lo;
  a.hi_val = act.hi_val;
  a.packed = packed;
  if (pack && pack_by_bytes(p, a.hl, sentinel)) {
    const dim3 grid((p.M * a.row_bytes + kThreads - 1) / kThreads);
    if (sentinel) hipLaunchKernelGGL(pack_bytes_kernel<true>, grid, dim3(kThreads), 0, st, a);
    else hipLaunchKernelGGL(pack_bytes_kernel<false>, grid, dim3(kThreads), 0, st, a);
    return hipGetLastError() == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
  }
  // Enough rows for every thread to have 32 channels: rows of 8192 channels and more go one by one.  The longest row is
  // 48 KB (65536 channels), below the default limit of dynamic LDS.  Where that leaves half of the compute units without work,
  // packing takes half as many rows at a time (sentinel [1016,320] 4.5 -> 3.3 us).
  constexpr int kChannels = 32 * kThreads;
  const int cus = device_compute_units();
  a.rows = (kChannels + p.K - 1) / p.K;
  if (pack && (p.M + a.rows - 1) / a.rows <= cus / 2) a.rows = (kChannels / 2 + p.K - 1) / p.K;
  const size_t lds = static_cast<size_t>(a.rows) * a.row_bytes + 48;  // the offset in front, and what a 64-bit read passes
  const dim3 grid(static_cast<unsigned>((static_cast<int64_t>(p.M) + a.rows - 1) / a.rows));
  // Longer rows take twice the threads ([64,16384] packs in 3.9 us instead of 5.1, unpacks in 4.2 instead of 5.4); packing many
  // of them does not ([4096,11008] 22.4 instead of 21.6 us).
  const bool wide = p.K > kChannels && (!pack || p.M <= 2 * cus);
#define SQ_LAUNCH(KERNEL, SENTINEL)                                                                                      \
  if (wide) hipLaunchKernelGGL((KERNEL<2 * kThreads, SENTINEL>), grid, dim3(2 * kThreads), lds, st, a);                 \
  else hipLaunchKernelGGL((KERNEL<kThreads, SENTINEL>), grid, dim3(kThreads), lds, st, a)
  if (pack && sentinel) { SQ_LAUNCH(pack_storage_kernel, true); }
  else if (pack) { SQ_LAUNCH(pack_storage_kernel, false); }
  else if (sentinel) { SQ_LAUNCH(unpack_storage_kernel, true); }
  else { SQ_LAUNCH(unpack_storage_kernel, false); }
#undef SQ_LAUNCH
  return hipGetLastError() == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}

}  // namespace sq
