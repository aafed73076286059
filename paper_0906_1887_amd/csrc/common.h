// Internal helpers shared by the libcorr kernels and host code (not part of
// the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace corr {

// Workgroups are handed to the 8 XCDs of an MI355X round-robin by workgroup
// id, and each XCD has its own L2.  Kernels remap blockIdx.x so that a
// contiguous range of work items (e.g. all baseline tiles of one channel,
// which re-read the same input rows) runs on one XCD, in order.
constexpr int kNumXcd = 8;

// Element kinds of the matrix-core X-engine.
constexpr int kElemI8 = 0;
constexpr int kElemF16 = 1;
constexpr int kElemF8 = 2;
constexpr int kElemCI4 = 3;   // int8 engine on 4-bit complex samples, one byte each
constexpr int kElemF16Cvt = 4;  // FP16 engine converting complex float32 as it stages
constexpr int kElemF8Cvt = 5;   // FP8 engine converting (with the per-channel scale) as it stages
constexpr int kElemF32 = 6;     // complex float32 on v_mfma_f32_16x16x4_f32 (64-row tiles)

__device__ __forceinline__ int64_t xcd_item(int64_t bid, int64_t per_xcd) {
  const int64_t xcd = bid % kNumXcd;
  const int64_t slot = bid / kNumXcd;
  return xcd * per_xcd + slot;
}

// Lower-triangle tile (I >= J) of linear index t = I(I+1)/2 + J.
__device__ __forceinline__ void tile_decode(int t, int& I, int& J) {
  int i = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
  while (i * (i + 1) / 2 > t) --i;
  while ((i + 1) * (i + 2) / 2 <= t) ++i;
  I = i;
  J = t - i * (i + 1) / 2;
}

// sizeof(V) bytes from an address of any alignment, as one load (global memory
// takes unaligned loads on gfx950 under this ABI).
template <typename V>
__device__ __forceinline__ V load_any(const void* p) {
  V v;
  __builtin_memcpy(&v, p, sizeof(V));
  return v;
}
template <typename V>
__device__ __forceinline__ V load16_any(const void* p) {
  static_assert(sizeof(V) == 16, "16 bytes");
  return load_any<V>(p);
}

__device__ __forceinline__ int64_t tri_index(int64_t i, int64_t j) { return i * (i + 1) / 2 + j; }

// Triangle index of (i + d, 0) for small constants d, from that of (i, 0): one
// full multiplication for a block of rows instead of one a product (a 32-bit
// one takes four times as long as a 24-bit one), which is half a microsecond of
// every launch with few inputs.
struct TriRow {
  uint32_t i, t;
  __device__ __forceinline__ explicit TriRow(int row) : i((uint32_t)row), t(i * (i + 1) / 2) {}   // i < 65536
  __device__ __forceinline__ uint32_t at(int d) const {
    return t + (uint32_t)__umul24(i, (uint32_t)d) + (uint32_t)(d * (d + 1) / 2);
  }
};

// Adds N products v[k] to out[off[k]] (kNoProduct: none).  Every old value is
// loaded before the first sum is stored: one product at a time, each load waits
// behind the stores before it.  Later passes of an integration, 256 inputs x 512
// channels x 512 samples: int8 124 -> 92 us, CI4 112 -> 79, FP16 283 -> 222; 355 x
// 264 x 88: FP16 156 -> 115, FP8 247 -> 189; 1024 x 64 x 512 int8 259 -> 173.
// Two engines still add one product at a time: the unaligned int8 one, whose
// 128-row tile has no register to spare for it (22 spills), and the plain FP32
// one, where it was not tried.
constexpr uint32_t kNoProduct = 0xFFFFFFFFu;
template <typename V, int N>
__device__ __forceinline__ void add_products(V* __restrict__ out, const uint32_t (&off)[N], const V (&v)[N]) {
  V o[N];
#pragma unroll
  for (int k = 0; k < N; ++k) o[k] = out[off[k] != kNoProduct ? off[k] : 0];
#pragma unroll
  for (int k = 0; k < N; ++k)
    if (off[k] != kNoProduct) {
      o[k].x += v[k].x;
      o[k].y += v[k].y;
      out[off[k]] = o[k];
    }
}
template <typename V, int N>
__device__ __forceinline__ void put_products(V* __restrict__ out, const uint32_t (&off)[N], const V (&v)[N],
                                             int accumulate) {
  if (accumulate) {
    add_products(out, off, v);
  } else {
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (off[k] != kNoProduct) out[off[k]] = v[k];
  }
}

// The same of products value(k) for out[index(k)], those for which in(k) holds,
// each made only where it is stored, unless they are added (faster where a wave
// holds many blocks: 121 inputs x 7 channels x 220 samples on staged FP16 rows,
// the kernel 12.7 -> 11.2 us; the converting kernels spill with it).
template <typename V, int N, class In, class Index, class Value>
__device__ __forceinline__ void put_each(V* __restrict__ out, In in, Index index, Value value, int accumulate) {
  if (accumulate) {
    uint32_t off[N];
    V v[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
      off[k] = in(k) ? index(k) : kNoProduct;
      v[k] = value(k);
    }
    add_products(out, off, v);
  } else {
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (in(k)) out[index(k)] = value(k);
  }
}

// Kernel argument block of the X-engines.
struct XArgs {
  const void* x;            // samples [n_ch][n_in][row_stride] (complex)
  int64_t row_stride_b;     // bytes between consecutive input rows
  int64_t ch_stride_b;      // bytes between channels
  int64_t k_bytes;          // valid bytes per row (n_samples * bytes per sample)
  int64_t k_split_bytes;    // bytes per K split (multiple of the K chunk)
  void* out;                // accumulator [n_ch][P][2] (or split partials)
  int64_t out_split_stride; // elements between split partial buffers
  int64_t n_products;       // P
  int32_t n_in;
  int32_t n_ch;
  int32_t n_tiles;          // lower-triangle tiles per channel
  int32_t n_split;          // K splits
  int32_t n_items;          // workgroups with work: channels x tiles x splits for the engines that take one tile
                            // each (item_decode); plain FP32 pairs diagonal tiles or takes several channels, and
                            // the one-workgroup FP16 kernel has channels x splits
  int32_t per_xcd;          // ceil(n_items / 8)
  int32_t accumulate;       // 1: out += tile; 0: out = tile
  int32_t pad_;
  const float* inv_scale2;  // FP8: per-channel 1/s_c^2 applied in the epilogue (else null)
  const uint32_t* m_bits;   // converting FP8 engine: per-channel max |re|, |im| (float bits)
};

// Work item -> (channel, K split, tile I >= J) of the matrix-core engines:
// tile fastest, then split, then channel, so that a channel's tiles (which
// share its row panels) start together on one XCD (xcd_item keeps each XCD's
// items contiguous).  An order that ran each XCD's off-diagonal tiles before
// its diagonal ones read less from HBM on C3 but was measured slower there
// (1.5 %) and on the FP16 engine (10 %), so it was removed.
__device__ __forceinline__ void item_decode(const XArgs& a, int64_t item, int& ch, int& split, int& I, int& J) {
  const int tile = (int)(item % a.n_tiles);
  const int64_t rest = item / a.n_tiles;
  split = (int)(rest % a.n_split);
  ch = (int)(rest / a.n_split);
  tile_decode(tile, I, J);
}

// FP8 scale of a channel with max |re|, |im| = m: the largest power of two s
// with s * m <= 448 (the largest finite E4M3 value); 1 when m is 0 or not
// finite.  The exponent is kept in [-60, 60] (so 1/s^2 stays a normal float)
// and the correction loops are bounded; within that range the result is
// exact, because s is a power of two and the comparisons are exact.
__device__ __forceinline__ float e4m3_scale(float m) {
  if (!(m > 0.f) || !(m < INFINITY)) return 1.f;
  const float e = fminf(fmaxf(floorf(log2f(448.f / m)), -60.f), 60.f);
  float s = ldexpf(1.f, (int)e);
  for (int k = 0; k < 4 && s * m > 448.f && s > 0x1p-60f; ++k) s *= 0.5f;
  for (int k = 0; k < 4 && 2.f * s * m <= 448.f && s < 0x1p60f; ++k) s *= 2.f;
  return s;
}

}  // namespace corr
