// The SQ-format at its equivalent bit width (Section 4.1: y = (1-s)*h_high + s*h_low bits per element):
// conversion between the compute containers of an sq_act (INT8 high codes, 4-bit low codes dense over K)
// and the packed stream -- per token row the high codes of the high channels at h_high bits each, then the low
// codes of the low channels only at h_low bits each, ascending channel order, least significant bit first.
//
// Bound by HBM in both directions.  A workgroup converts a few whole rows (consecutive bytes of the stream) through an
// image of them in LDS: the image starts at the stream's own offset inside 16 bytes, so that whatever the length of a row
// the stream is read and written 16 bytes at a time, and bit fields of any width and place are ORed into, or cut out of,
// LDS dwords.  A thread converts 32 channels at a time.  With one thread per byte of the stream, which looked its channel
// up in the mask, [4096,4096] took 110 us to pack and 33 us to unpack, against 8.7 and 11.1 us.
#include "sq_gemm_common.h"

namespace sq {
namespace {

using gemm::v4u;

constexpr int NT = 256;

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

template <bool SENTINEL>
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

template <bool SENTINEL>
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
  // enough rows for every thread to have 32 channels: rows of 8192 channels and more go one by one.  The longest row is
  // 48 KB (65536 channels), below the default limit of dynamic LDS
  a.rows = p.K >= 32 * NT ? 1 : (32 * NT + p.K - 1) / p.K;
  const size_t lds = static_cast<size_t>(a.rows) * a.row_bytes + 48;  // the offset in front, and what a 64-bit read passes
  const dim3 grid(static_cast<unsigned>((static_cast<int64_t>(p.M) + a.rows - 1) / a.rows));
  if (pack && sentinel) hipLaunchKernelGGL(pack_storage_kernel<true>, grid, dim3(NT), lds, st, a);
  else if (pack) hipLaunchKernelGGL(pack_storage_kernel<false>, grid, dim3(NT), lds, st, a);
  else if (sentinel) hipLaunchKernelGGL(unpack_storage_kernel<true>, grid, dim3(NT), lds, st, a);
  else hipLaunchKernelGGL(unpack_storage_kernel<false>, grid, dim3(NT), lds, st, a);
  return hipGetLastError() == hipSuccess ? SQ_OK : SQ_ERR_LAUNCH;
}

}  // namespace sq
