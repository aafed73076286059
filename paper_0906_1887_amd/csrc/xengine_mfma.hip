// Matrix-core X-engine for aligned sample rows: int8 (int32 accumulation),
// FP16 and OCP FP8 E4M3 (FP32 accumulation).
//
// V_ij[c] += sum_t x_i[c,t] conj(x_j[c,t]) -- the cross-multiply-accumulate
// of Sec. 4 (third step), per channel, over the lower-triangle baseline tiles
// of Fig. 2's outer product.  Each input row holds interleaved (re, im)
// elements along K = 2T, so per channel
//     Re V = A B^T            Im V = A (iB)^T,  iB = (-im_j, re_j)
// and iB is formed from the staged B fragment in registers (a byte or
// half-word rotation with a sign flip), so one LDS read feeds both products.
//
// Pipeline: a workgroup (4 waves, 2 x 2) owns a BT x BT tile of one channel.
// Operand rows are staged 64 K-bytes at a time straight from global memory
// into LDS (global_load_lds_dwordx4: no registers, no VALU), NS stages deep,
// so loads for stage s+NS-1 are in flight while stage s feeds the MFMAs; one
// barrier per stage.  LDS rows are 64 bytes with the four 16-byte chunks
// XOR-permuted by row so that the 32 rows of an MFMA fragment read hit
// distinct banks.  Rows past N_I are loaded from a clamped address and only
// ever reach outputs that are never stored; bytes past the valid K range are
// zeroed in LDS before use.  Tiles are numbered channel-major and remapped
// from blockIdx.x so that each XCD (and its L2) runs a contiguous range of
// channels.
#include <type_traits>

#include "common.h"
#include "launch.h"

namespace corr {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

constexpr int kMKC = 64;   // K bytes per stage
constexpr int kMNS = 4;    // pipeline stages

// 16-byte chunk c (0..3) of LDS row r lives at chunk c ^ swz(r).
__device__ __forceinline__ int swz(int r) { return (r >> 2) & 3; }

// Multiply packed complex elements by i: (re, im) -> (-im, re).
__device__ __forceinline__ int rot_i8(int w) {
  const uint32_t u = (uint32_t)w;
  const uint32_t im = (u >> 8) & 0x00FF00FFu;
  const uint32_t neg = 0x01000100u - im;            // low byte of each 16-bit lane = -im
  return (int)((neg & 0x00FF00FFu) | ((u << 8) & 0xFF00FF00u));
}
__device__ __forceinline__ int rot_f16(int w) {     // one complex half pair per dword
  const uint32_t u = (uint32_t)w;
  return (int)(((u >> 16) ^ 0x8000u) | (u << 16));
}
__device__ __forceinline__ int rot_f8(int w) {      // two complex fp8 pairs per dword
  const uint32_t u = (uint32_t)w;
  const uint32_t sw = ((u >> 8) & 0x00FF00FFu) | ((u << 8) & 0xFF00FF00u);
  return (int)(sw ^ 0x00800080u);
}

template <int EK>
__device__ __forceinline__ v4i rot4(v4i v) {
  v4i r;
  if constexpr (EK == kElemF32) {   // two complex float32 per 16 bytes: (re, im) -> (-im, re)
    r[0] = (int)((uint32_t)v[1] ^ 0x80000000u);
    r[1] = v[0];
    r[2] = (int)((uint32_t)v[3] ^ 0x80000000u);
    r[3] = v[2];
    return r;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
    r[q] = EK == kElemI8 ? rot_i8(v[q]) : (EK == kElemF16 ? rot_f16(v[q]) : rot_f8(v[q]));
  return r;
}

// CI4 samples (one byte per complex sample: re in bits 7..4, im in bits 3..0,
// two's complement nibbles, the "1-byte" mode of Sec. 5) are unpacked in
// registers into int8 operands scaled by 16: the byte's high nibble with the
// low nibble cleared is 16 re, and the low nibble shifted up is 16 im, both
// exact in int8 for |re|, |im| <= 7.  Operand bytes run [16 re of 4 samples,
// 16 im of the same 4, 16 re of the next 4, 16 im of those]; the same order
// in A and B makes A B^T = sum (re re' + im im') = Re V (times 256).
constexpr uint32_t kHiNib = 0xF0F0F0F0u;
__device__ __forceinline__ v4i ci4_plain(int w0, int w1) {
  const uint32_t u0 = (uint32_t)w0, u1 = (uint32_t)w1;
  return v4i{(int)(u0 & kHiNib), (int)((u0 << 4) & kHiNib), (int)(u1 & kHiNib), (int)((u1 << 4) & kHiNib)};
}
// -16 re per byte of a high-nibble word: flip the nibble and add 1 in it; a
// carry out of a byte (re = 0) lands in the next byte's clear low nibble and
// is masked off.
__device__ __forceinline__ uint32_t neg_hi_nibbles(uint32_t x) { return ((x ^ kHiNib) + 0x10101010u) & kHiNib; }
// Operands of -iA = (im, -re) in the same byte order: A' B^T = sum (im re' -
// re im') = Im V (times 256).
__device__ __forceinline__ v4i ci4_rotm(int w0, int w1) {
  const uint32_t u0 = (uint32_t)w0, u1 = (uint32_t)w1;
  return v4i{(int)((u0 << 4) & kHiNib), (int)neg_hi_nibbles(u0 & kHiNib), (int)((u1 << 4) & kHiNib),
             (int)neg_hi_nibbles(u1 & kHiNib)};
}

template <int EK>
struct MAcc;
template <>
struct MAcc<kElemI8> { typedef v16i T; };
template <>
struct MAcc<kElemCI4> { typedef v16i T; };
template <>
struct MAcc<kElemF16> { typedef v16f T; };
template <>
struct MAcc<kElemF8> { typedef v16f T; };

// One 64-byte K stage of a 32 x 32 block: fragments are two 16-byte reads per
// lane (K bytes g*16.. and 32+g*16.., g = lane / 32) of A and of B.
template <int EK>
__device__ __forceinline__ void mfma64(const v4i (&a)[2], const v4i (&b)[2], typename MAcc<EK>::T& acc) {
  if constexpr (EK == kElemI8) {
    acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[0], b[0], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[1], b[1], acc, 0, 0, 0);
  } else if constexpr (EK == kElemF16) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a[0]), __builtin_bit_cast(v8h, b[0]),
                                                  acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a[1]), __builtin_bit_cast(v8h, b[1]),
                                                  acc, 0, 0, 0);
  } else {
    const v8i a8 = {a[0][0], a[0][1], a[0][2], a[0][3], a[1][0], a[1][1], a[1][2], a[1][3]};
    const v8i b8 = {b[0][0], b[0][1], b[0][2], b[0][3], b[1][0], b[1][1], b[1][2], b[1][3]};
    // format 0 (FP8 E4M3) for both operands, unit E8M0 scales (127 = 2^0)
    acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, acc, 0, 0, 0, 127, 0, 127);
  }
}

// The same of packed CI4 samples: each read holds 16, of two K halves.  Up to 64
// inputs in 64-row tiles: 32 x 90 channels x 7109 samples to dump 36 us, 60 in
// 128-row tiles (16 times the products that are stored); 64 x 512 x 4000 54 and
// 115.
__device__ __forceinline__ void mfma64_ci4(const v4i (&a)[2], const v4i (&b)[2], v16i& vr, v16i& vi) {
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int q = 0; q < 4; q += 2) {
      const v4i bp = ci4_plain(b[h][q], b[h][q + 1]);
      vr = __builtin_amdgcn_mfma_i32_32x32x32_i8(ci4_plain(a[h][q], a[h][q + 1]), bp, vr, 0, 0, 0);
      vi = __builtin_amdgcn_mfma_i32_32x32x32_i8(ci4_rotm(a[h][q], a[h][q + 1]), bp, vi, 0, 0, 0);
    }
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

template <int EK, int BT, bool DIAG>
__device__ __forceinline__ void mfma_tile(const XArgs& a, int8_t* lds, int ch, int split, int I, int J) {
  constexpr int WT = BT / 2;                 // wave tile
  constexpr int MB = WT / 32;                // 32 x 32 blocks per wave side
  constexpr int PANEL = BT * kMKC;           // bytes per operand per stage
  constexpr int STAGE = PANEL * (DIAG ? 1 : 2);
  constexpr int QPW = BT / 16 / 4;           // 1 KB load instructions per operand per wave
  constexpr int LPW = QPW * (DIAG ? 1 : 2);  // load instructions per wave per stage
  using Acc = typename MAcc<EK>::T;

  const int8_t* __restrict__ xc = static_cast<const int8_t*>(a.x) + (int64_t)ch * a.ch_stride_b;
  const int64_t k0 = (int64_t)split * a.k_split_bytes;
  const int64_t k1 = min(a.k_bytes, k0 + a.k_split_bytes);
  const int n_st = k1 > k0 ? (int)((k1 - k0 + kMKC - 1) / kMKC) : 0;
  const int64_t last = ((k1 - 1) >> 4) << 4;  // last valid 16-byte chunk start

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const bool wave_idle = DIAG && (wm < wn);

  // This lane's part of each load instruction: LDS row lrow (of 16), chunk p.
  const int lrow = lane >> 2, p = lane & 3;
  const int8_t* gA[QPW];
  const int8_t* gB[QPW];
  int rowq[QPW];
#pragma unroll
  for (int q = 0; q < QPW; ++q) {
    const int r = (wave * QPW + q) * 16 + lrow;    // tile row
    rowq[q] = r;
    const int c = p ^ swz(r);                      // global chunk this lane fetches
    const int ra = min(I * BT + r, a.n_in - 1);
    gA[q] = xc + (int64_t)ra * a.row_stride_b + 16 * c;
    if (!DIAG) {
      const int rb = min(J * BT + r, a.n_in - 1);
      gB[q] = xc + (int64_t)rb * a.row_stride_b + 16 * c;
    }
  }

  auto issue = [&](int st) {
    int8_t* base = lds + (st % kMNS) * STAGE;
    const int64_t kb = k0 + (int64_t)st * kMKC;
#pragma unroll
    for (int q = 0; q < QPW; ++q) {
      const int c = p ^ swz(rowq[q]);
      const int64_t kk = kb + 16 * c;
      const int64_t off = (kk <= last ? kb : last - 16 * c);   // keep the 16 bytes inside the row
      int8_t* dst = base + (wave * QPW + q) * 1024;
      __builtin_amdgcn_global_load_lds(gA[q] + off, dst, 16, 0, 0);
      if (!DIAG) __builtin_amdgcn_global_load_lds(gB[q] + off, dst + PANEL, 16, 0, 0);
    }
  };
  // Zero / mask the chunks of stage st that reach past k1 (only the last stage).
  auto fix_tail = [&](int st) {
    int8_t* base = lds + (st % kMNS) * STAGE;
    const int64_t kb = k0 + (int64_t)st * kMKC;
#pragma unroll
    for (int q = 0; q < QPW; ++q) {
      const int c = p ^ swz(rowq[q]);
      const int64_t kk = kb + 16 * c;
      if (kk + 16 > k1) {
        const int64_t valid = k1 - kk;
#pragma unroll
        for (int op = 0; op < (DIAG ? 1 : 2); ++op) {
          v4i* cell = reinterpret_cast<v4i*>(base + op * PANEL + (wave * QPW + q) * 1024 + lane * 16);
          v4i v = *cell;
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const int64_t lo = 4 * w;
            const int keep = valid >= lo + 4 ? 4 : (valid > lo ? (int)(valid - lo) : 0);
            const uint32_t m = keep >= 4 ? 0xFFFFFFFFu : ((1u << (8 * keep)) - 1u);
            v[w] = (int)((uint32_t)v[w] & m);
          }
          *cell = v;
        }
      }
    }
  };

  Acc vr[MB][MB], vi[MB][MB];
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < MB; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        vr[m][n][r] = 0;
        vi[m][n][r] = 0;
      }

#pragma unroll
  for (int s = 0; s < kMNS - 1; ++s)
    if (s < n_st) issue(s);

  const int frow = lane & 31;
  const int g = lane >> 5;
  const bool tail = (k1 - k0) % kMKC != 0;
  for (int s = 0; s < n_st; ++s) {
    // Wait for this wave's loads of stage s; later stages may stay in flight.
    const int ahead = min(kMNS - 2, n_st - 1 - s);
    if (ahead >= 2) wait_vmcnt<2 * LPW>();
    else if (ahead == 1) wait_vmcnt<LPW>();
    else wait_vmcnt<0>();
    if (tail && s == n_st - 1) {
      fix_tail(s);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    // Plain s_barrier (as asm with a memory clobber, so the compiler keeps
    // LDS reads below it): each wave has already waited for its own stage-s
    // loads, which is all the other waves need; a fenced barrier would also
    // drain the loads of later stages that are meant to stay in flight.
    asm volatile("s_barrier" ::: "memory");
    if (s + kMNS - 1 < n_st) issue(s + kMNS - 1);
    if (!wave_idle) {
      const int8_t* As = lds + (s % kMNS) * STAGE;
      const int8_t* Bs = DIAG ? As : As + PANEL;
      v4i af[MB][2], bf[MB][2], bj[MB][2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int cidx = 2 * h + g;            // logical 16-byte chunk
#pragma unroll
        for (int m = 0; m < MB; ++m) {
          const int r = wm * WT + m * 32 + frow;
          af[m][h] = *reinterpret_cast<const v4i*>(As + r * kMKC + 16 * (cidx ^ swz(r)));
        }
#pragma unroll
        for (int n = 0; n < MB; ++n) {
          const int r = wn * WT + n * 32 + frow;
          bf[n][h] = *reinterpret_cast<const v4i*>(Bs + r * kMKC + 16 * (cidx ^ swz(r)));
          if constexpr (EK != kElemCI4) bj[n][h] = rot4<EK>(bf[n][h]);
        }
      }
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < MB; ++n) {
          if (DIAG && wm == wn && m < n) continue;   // strictly upper 32 x 32 block
          if constexpr (EK == kElemCI4) {
            mfma64_ci4(af[m], bf[n], vr[m][n], vi[m][n]);
          } else {
            mfma64<EK>(af[m], bf[n], vr[m][n]);
            mfma64<EK>(af[m], bj[n], vi[m][n]);
          }
        }
    }
  }

  if (wave_idle) return;
  // Epilogue.  32 x 32 accumulator layout: register r of lane l holds row
  // 8*(r/4) + 4*(l/32) + r%4, column l%32.
  float scale = 1.0f;
  if constexpr (EK == kElemF8) scale = a.inv_scale2 ? a.inv_scale2[ch] : 1.0f;
  auto scaled = [&](auto x) {
    if constexpr (EK == kElemI8) return x;
    else if constexpr (EK == kElemCI4) return x >> 8;   // the operands are 16 x the sample parts
    else return x * scale;
  };
  const int64_t out0 = (int64_t)split * a.out_split_stride + (int64_t)ch * a.n_products;
  // Few inputs: rows past the last one are passed by, and indexes come from one
  // multiplication.  The kernel on 2 inputs x 18 channels x 5112 samples FP16 in
  // three chunks 6.84 -> 6.40 us, 10 x 21 x 116 5.96 -> 5.36.  Not for the others: CI4
  // and FP8 lose up to 5 % at 17 to 64 inputs with it, int8 5 us of a pass of 64
  // inputs x 128 channels x 10000 samples.
  constexpr bool kFew = EK == kElemF16;
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < MB; ++n) {
      if (DIAG && wm == wn && m < n) continue;
      const int j = J * BT + wn * WT + n * 32 + (lane & 31);
      const int i0 = I * BT + __builtin_amdgcn_readfirstlane(wm) * WT + m * 32;
      const TriRow row(i0 + 4 * (lane >> 5));
#pragma unroll
      for (int h = 0; h < 16; h += 8) {
        if (kFew && i0 + 2 * h >= a.n_in) break;   // rows past the last input
        uint32_t off[8];
        std::conditional_t<std::is_same_v<Acc, v16i>, int2, float2> v[8];
#pragma unroll
        for (int r = h; r < h + 8; ++r) {
          const int d = 8 * (r >> 2) + (r & 3);
          const int i = (int)row.i + d;
          off[r - h] = i < a.n_in && j <= i ? (kFew ? row.at(d) + (uint32_t)j : (uint32_t)tri_index(i, j)) : kNoProduct;
          v[r - h].x = scaled(vr[m][n][r]);
          v[r - h].y = i == j ? 0 : scaled(vi[m][n][r]);
        }
        put_products(static_cast<std::remove_reference_t<decltype(v[0])>*>(a.out) + out0, off, v, a.accumulate);
      }
    }
}

// Multiply packed complex elements by -i: (re, im) -> (im, -re).
__device__ __forceinline__ int rotm_i8(int w) {
  const uint32_t u = (uint32_t)w;
  const uint32_t neg = 0x01000100u - (u & 0x00FF00FFu);   // low byte of each 16-bit lane = -re
  // bytes: im0 (u.1), -re0 (neg.0), im1 (u.3), -re1 (neg.2)
  return (int)__builtin_amdgcn_perm(neg, u, 0x06030401u);
}
__device__ __forceinline__ int rotm_f16(int w) {
  const uint32_t u = (uint32_t)w;
  return (int)(((u >> 16) | (u << 16)) ^ 0x80000000u);
}
__device__ __forceinline__ int rotm_f8(int w) {
  const uint32_t u = (uint32_t)w;
  const uint32_t sw = ((u >> 8) & 0x00FF00FFu) | ((u << 8) & 0xFF00FF00u);
  return (int)(sw ^ 0x80008000u);
}

template <int EK>
__device__ __forceinline__ v4i rotm4(v4i v) {
  v4i r;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    r[q] = EK == kElemI8 ? rotm_i8(v[q]) : (EK == kElemF16 ? rotm_f16(v[q]) : rotm_f8(v[q]));
  return r;
}

// One 32 x 32 block product over 16 K bytes per lane (int8: K = 32, FP16:
// K = 16).  FP8 blocks take both 16-byte halves at once (mfma64).
template <int EK>
__device__ __forceinline__ void mfma16(const v4i& a, const v4i& b, typename MAcc<EK>::T& acc) {
  static_assert(EK != kElemF8, "FP8 products span 32 K bytes per lane");
  if constexpr (EK == kElemI8) {
    acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, acc, 0, 0, 0);
  } else {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), acc, 0, 0, 0);
  }
}

// 128 x 128 tile, four waves (2 x 2) of 64 x 64, two workgroups per CU so
// that each SIMD holds two waves.  Per stage a wave reads 8 fragments (A and
// B, two 32-row blocks each, two K halves) and issues 16 MFMAs (8 for FP8).
// Fragments are double-buffered in registers: the LDS reads of stage s+1 are
// interleaved with the MFMAs of stage s.  The barrier of stage s+1 follows
// every wave's completed reads of stage s, so stage s+NS may then be loaded
// into stage s's buffer.  Loads of stages that lie wholly inside the K range
// use uniform tile bases and 32-bit per-lane offsets (LDS destinations in
// scalar registers); the last stage clamps its addresses and is masked.
template <int EK, bool DIAG>
__device__ __forceinline__ void mfma_tile_128(const XArgs& a, int8_t* lds, int ch, int split, int I, int J) {
  constexpr int BT = 128;
  constexpr int PANEL = BT * kMKC;           // bytes per operand per stage
  constexpr int STAGE = PANEL * (DIAG ? 1 : 2);
  constexpr int QPW = BT / 16 / 4;           // 1 KB load instructions per operand per wave
  constexpr int LPW = QPW * (DIAG ? 1 : 2);  // load instructions per wave per stage
  constexpr int NMF = EK == kElemF8 ? 8 : 16;  // MFMAs per wave per stage
  using Acc = typename MAcc<EK>::T;

  const int8_t* __restrict__ xc = static_cast<const int8_t*>(a.x) + (int64_t)ch * a.ch_stride_b;
  const int64_t k0 = (int64_t)split * a.k_split_bytes;
  const int64_t k1 = min(a.k_bytes, k0 + a.k_split_bytes);
  const int n_st = k1 > k0 ? (int)((k1 - k0 + kMKC - 1) / kMKC) : 0;
  const int64_t last = ((k1 - 1) >> 4) << 4;   // last valid 16-byte chunk start
  // Stages whose 64 bytes all lie in [k0, k1) and whose offsets fit 32 bits.
  const int n_fast = a.row_stride_b < (int64_t(1) << 24) ? (int)((k1 - k0) / kMKC) : 0;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  // This lane's part of each load instruction: LDS row lrow (of 16), chunk p.
  const int lrow = lane >> 2, p = lane & 3;
  const int8_t* gA[QPW];
  const int8_t* gB[QPW];
  uint32_t oA[QPW], oB[QPW];
  int rowq[QPW];
  const int8_t* tA = xc + (int64_t)(I * BT) * a.row_stride_b + k0;
  const int8_t* tB = xc + (int64_t)(J * BT) * a.row_stride_b + k0;
#pragma unroll
  for (int q = 0; q < QPW; ++q) {
    const int r = (wave * QPW + q) * 16 + lrow;    // tile row
    rowq[q] = r;
    const int c = p ^ swz(r);                      // global chunk this lane fetches
    const int ra = min(I * BT + r, a.n_in - 1);
    const int rb = min(J * BT + r, a.n_in - 1);
    gA[q] = xc + (int64_t)ra * a.row_stride_b + 16 * c;
    gB[q] = xc + (int64_t)rb * a.row_stride_b + 16 * c;
    oA[q] = (uint32_t)((int64_t)(ra - I * BT) * a.row_stride_b + 16 * c);
    oB[q] = (uint32_t)((int64_t)(rb - J * BT) * a.row_stride_b + 16 * c);
  }
  auto issue = [&](int st) {
    int8_t* base = lds + (st % kMNS) * STAGE + wave * QPW * 1024;
    if (st < n_fast) {
      const int8_t* ga = tA + st * kMKC;
      const int8_t* gb = tB + st * kMKC;
#pragma unroll
      for (int q = 0; q < QPW; ++q) {
        __builtin_amdgcn_global_load_lds(ga + oA[q], base + q * 1024, 16, 0, 0);
        if (!DIAG) __builtin_amdgcn_global_load_lds(gb + oB[q], base + q * 1024 + PANEL, 16, 0, 0);
      }
    } else {
      const int64_t kb = k0 + (int64_t)st * kMKC;
#pragma unroll
      for (int q = 0; q < QPW; ++q) {
        const int c = p ^ swz(rowq[q]);
        const int64_t kk = kb + 16 * c;
        const int64_t off = (kk <= last ? kb : last - 16 * c);   // keep the 16 bytes inside the row
        __builtin_amdgcn_global_load_lds(gA[q] + off, base + q * 1024, 16, 0, 0);
        if (!DIAG) __builtin_amdgcn_global_load_lds(gB[q] + off, base + q * 1024 + PANEL, 16, 0, 0);
      }
    }
  };
  // Zero / mask the chunks of stage st that reach past k1 (only the last stage).
  auto fix_tail = [&](int st) {
    int8_t* base = lds + (st % kMNS) * STAGE;
    const int64_t kb = k0 + (int64_t)st * kMKC;
#pragma unroll
    for (int q = 0; q < QPW; ++q) {
      const int c = p ^ swz(rowq[q]);
      const int64_t kk = kb + 16 * c;
      if (kk + 16 > k1) {
        const int64_t valid = k1 - kk;
#pragma unroll
        for (int op = 0; op < (DIAG ? 1 : 2); ++op) {
          v4i* cell = reinterpret_cast<v4i*>(base + op * PANEL + (wave * QPW + q) * 1024 + lane * 16);
          v4i v = *cell;
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const int64_t lo = 4 * w;
            const int keep = valid >= lo + 4 ? 4 : (valid > lo ? (int)(valid - lo) : 0);
            const uint32_t m = keep >= 4 ? 0xFFFFFFFFu : ((1u << (8 * keep)) - 1u);
            v[w] = (int)((uint32_t)v[w] & m);
          }
          *cell = v;
        }
      }
    }
  };

  Acc vr[2][2], vi[2][2];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        vr[m][n][r] = 0;
        vi[m][n][r] = 0;
      }

#pragma unroll
  for (int s = 0; s < kMNS - 1; ++s)
    if (s < n_st) issue(s);

  const int frow = lane & 31;
  const int g = lane >> 5;
  const bool tail = (k1 - k0) % kMKC != 0;
  // Wait for this wave's loads of stage st (later stages stay in flight),
  // mask the K tail, and make stage st visible to all waves.  A plain
  // s_barrier: a fenced one would also drain the later stages' loads.
  auto arrive = [&](int st) {
    const int ahead = min(kMNS - 2, n_st - 1 - st);
    if (ahead >= 2) wait_vmcnt<2 * LPW>();
    else if (ahead == 1) wait_vmcnt<LPW>();
    else wait_vmcnt<0>();
    if (tail && st == n_st - 1) fix_tail(st);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    asm volatile("s_barrier" ::: "memory");
  };
  auto read = [&](int st, v4i (&af)[2][2], v4i (&bf)[2][2]) {
    const int8_t* As = lds + (st % kMNS) * STAGE;
    const int8_t* Bs = DIAG ? As : As + PANEL;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int cidx = 2 * h + g;              // logical 16-byte chunk
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const int r = wm * 64 + m * 32 + frow;
        af[m][h] = *reinterpret_cast<const v4i*>(As + r * kMKC + 16 * (cidx ^ swz(r)));
      }
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const int r = wn * 64 + n * 32 + frow;
        bf[n][h] = *reinterpret_cast<const v4i*>(Bs + r * kMKC + 16 * (cidx ^ swz(r)));
      }
    }
  };
  // Re products first; the -i rotation of A runs on the VALU while they
  // execute, then the Im products: Im V = (-iA) B^T.  Consecutive MFMAs go to
  // different accumulators.  SK: a diagonal wave of a diagonal tile skips its
  // strictly upper block (m 0, n 1).
  auto compute = [&](auto sk, const v4i (&af)[2][2], const v4i (&bf)[2][2]) {
    constexpr bool SK = decltype(sk)::value;
    v4i ra[2][2];
    if constexpr (EK == kElemF8) {
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n)
          if (!(SK && m == 0 && n == 1)) mfma64<EK>(af[m], bf[n], vr[m][n]);
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int h = 0; h < 2; ++h) ra[m][h] = rotm4<EK>(af[m][h]);
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n)
          if (!(SK && m == 0 && n == 1)) mfma64<EK>(ra[m], bf[n], vi[m][n]);
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
          for (int n = 0; n < 2; ++n)
            if (!(SK && m == 0 && n == 1)) mfma16<EK>(af[m][h], bf[n][h], vr[m][n]);
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int h = 0; h < 2; ++h) ra[m][h] = rotm4<EK>(af[m][h]);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
          for (int n = 0; n < 2; ++n)
            if (!(SK && m == 0 && n == 1)) mfma16<EK>(ra[m][h], bf[n][h], vi[m][n]);
    }
  };

  if (n_st > 0) {
    arrive(0);
    if (kMNS - 1 < n_st) issue(kMNS - 1);
  }
  // In a diagonal tile the wave of the strictly upper 64 x 64 quarter only
  // loads its share of the panel and keeps the barriers.
  if (DIAG && wm < wn) {
    for (int s = 0; s + 1 < n_st; ++s) {
      arrive(s + 1);
      if (s + kMNS < n_st) issue(s + kMNS);
    }
    return;
  }
  auto run = [&](auto sk) {
    constexpr int NM = (DIAG && decltype(sk)::value) ? NMF * 3 / 4 : NMF;   // MFMAs per stage
    v4i af0[2][2], bf0[2][2], af1[2][2], bf1[2][2];
    if (n_st > 0) read(0, af0, bf0);
    for (int s = 0; s + 1 < n_st; ++s) {
      arrive(s + 1);
      if (s + kMNS < n_st) issue(s + kMNS);
      read(s + 1, af1, bf1);
      compute(sk, af0, bf0);
#pragma unroll
      for (int q = 0; q < (NM < 8 ? NM : 8); ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
      }
      if constexpr (NM > 8) __builtin_amdgcn_sched_group_barrier(0x008, NM - 8, 0);
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          af0[m][h] = af1[m][h];
          bf0[m][h] = bf1[m][h];
        }
    }
    if (n_st > 0) compute(sk, af0, bf0);
  };
  if (DIAG && wm == wn) run(std::true_type{});
  else run(std::false_type{});

  // Epilogue.  32 x 32 accumulator layout: register r of lane l holds row
  // 8*(r/4) + 4*(l/32) + r%4, column l%32.
  float scale = 1.0f;
  if constexpr (EK == kElemF8) scale = a.inv_scale2 ? a.inv_scale2[ch] : 1.0f;
  auto scaled = [&](auto x) {
    if constexpr (EK == kElemI8) return x;
    else return x * scale;
  };
  const int64_t out0 = (int64_t)split * a.out_split_stride + (int64_t)ch * a.n_products;
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const int j = J * BT + wn * 64 + n * 32 + (lane & 31);
      const int i0 = I * BT + __builtin_amdgcn_readfirstlane(wm) * 64 + m * 32;
      const TriRow row(i0 + 4 * (lane >> 5));
      auto at = [](int r) { return 8 * (r >> 2) + (r & 3); };
#pragma unroll
      for (int h = 0; h < 16; h += 8) {
        if (i0 + 2 * h >= a.n_in) break;       // rows past the last input
        using V = std::conditional_t<std::is_same_v<Acc, v16i>, int2, float2>;
        put_each<V, 8>(
            static_cast<V*>(a.out) + out0,
            [&](int k) { return (int)row.i + at(h + k) < a.n_in && j <= (int)row.i + at(h + k); },
            [&](int k) { return row.at(at(h + k)) + (uint32_t)j; },
            [&](int k) {
              V v;
              v.x = scaled(vr[m][n][h + k]);
              v.y = (int)row.i + at(h + k) == j ? 0 : scaled(vi[m][n][h + k]);
              return v;
            },
            a.accumulate);
      }
    }
}

// FP16 / FP8 engine reading complex float32 directly (plans without a
// staging chunk): the conversion of the staged engines moves into the load.
// A stage's float32 samples (FP16: 16 per row, 128 bytes; FP8: 32 per row,
// 256 bytes) are fetched with coalesced 16-byte loads (consecutive lanes read
// consecutive bytes of a row) into registers, PF stages ahead; each 16-byte
// load (two complex samples) is converted in registers (round to nearest
// even; FP8 after scaling by the channel's power of two s_c, saturating) and
// written to LDS in the staged engine's swizzled layout (8 bytes for FP16, 4
// for FP8).  The MFMA stage is that of mfma_tile_128, so the sums are those
// of the staged engine on the same codes.  Two LDS stage buffers, one
// barrier per stage, one 128-row workgroup per CU (the register prefetch takes
// the room of a second; cvt_waves below sets its wave count).  Samples past the
// pass are zero; rows past N_I are read from a clamped row and never stored.
//
// Up to 64 inputs run 64-row tiles (32 x 32 per wave), 4 (FP16) or 3 (FP8)
// workgroups per CU, where the 128-row tile loaded and converted its 64 or more
// missing rows too: 16 inputs x 674 channels x 1063 samples to dump 148 -> 43 us
// (FP16), 32 x 512 x 2000 172 -> 60, 64 x 512 x 2000 216 -> 130 (4.4 TB/s of
// samples); FP8 15 x 102 x 1814 76 -> 41, 64 x 512 x 2000 293 -> 215 with its pass
// for the maximum.
//
// With one tile per channel the steady loop has no condition around its loads,
// so that the compiler waits for the oldest stage only (with one it waits for
// every load in flight: 64 inputs as above 216 -> 155 us by this alone, 128 x 512 x
// 2000 303 -> 279).  With several tiles it gains nothing: they drift apart and
// miss the rows that they share in L2 (4.9 -> 8.1 GB from memory for 256 x 512 x
// 4096).
constexpr int kPF = 3;   // stages of float32 samples in flight per workgroup (FP8; FP16 takes 4)

// Two floats -> two binary16 (round to nearest even), the first in the low half.
__device__ __forceinline__ uint32_t pack_f16x2(float lo, float hi) {
  return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)lo) | ((uint32_t)__builtin_bit_cast(uint16_t, (_Float16)hi) << 16);
}

// NW waves per workgroup: 2 rows of NW / 2 waves, each wave a 64 x (256 / NW)
// part of the tile (32 x 32 blocks 2 x NBN).  In a diagonal tile a block whose
// columns lie above its rows is skipped, and a wave with no block left only
// converts and keeps the barriers.
template <int EK, int BT, bool DIAG, int NW>
__device__ __forceinline__ void mfma_tile_cvt(const XArgs& a, int8_t* lds, int ch, int split, int I, int J) {
  constexpr int EKM = EK == kElemF16Cvt ? kElemF16 : kElemF8;   // the MFMA stage's element kind
  static_assert(NW == 4 || NW == 8, "4 or 8 waves");
  constexpr int NT = NW * 64;                     // threads
  constexpr int NWN = NW / 2;                     // waves across the tile's columns
  constexpr int NBN = BT / 32 / NWN;              // 32-column blocks per wave
  constexpr int MB = BT / 64;                     // 32-row blocks per wave
  constexpr int PANEL = BT * kMKC;                // bytes per operand per stage
  constexpr int STAGE = PANEL * (DIAG ? 1 : 2);
  constexpr int NOP = DIAG ? 1 : 2;
  constexpr int SB = EKM == kElemF16 ? 4 : 2;     // staged bytes per complex sample
  constexpr int SPS = kMKC / SB;                  // samples per row per stage
  constexpr int NF = SPS / 2;                     // float4 (two samples) per row per stage
  constexpr int L = BT * NF / NT;                 // float4 per thread per operand per stage
  using Acc = typename MAcc<EKM>::T;
  // register stages in flight: FP16 holds 2 float4 per thread and operand per
  // stage, so 4 stages fit at two waves per SIMD (2.6 % faster on C4 than 3);
  // FP8 holds 8 and keeps kPF.
  constexpr int PF = EKM == kElemF16 ? 4 : kPF;

  const float* __restrict__ xc = reinterpret_cast<const float*>(static_cast<const int8_t*>(a.x) + (int64_t)ch * a.ch_stride_b);
  const int64_t k0 = (int64_t)split * a.k_split_bytes;
  const int64_t k1 = min(a.k_bytes, k0 + a.k_split_bytes);
  const int n_st = k1 > k0 ? (int)((k1 - k0 + kMKC - 1) / kMKC) : 0;
  const int64_t t0 = k0 / SB, t1 = k1 / SB;        // sample range of the pass
  const int64_t rsf = a.row_stride_b / 4;          // floats between rows (row_stride_b: float32 bytes)
  float sc = 1.f;
  if constexpr (EKM == kElemF8) sc = e4m3_scale(__uint_as_float(a.m_bits[ch]));

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / NWN, wn = wave % NWN;

  // This thread's loads: row q_row[q] (of 128), float4 f = q_f[q] of the
  // row's stage; LDS byte offset of the converted bytes within a panel.
  const float* src[2][L];
  int q_f[L], q_lds[L];
#pragma unroll
  for (int q = 0; q < L; ++q) {
    const int idx = tid + NT * q;
    const int r = idx / NF, f = idx % NF;
    const int kb = f * 2 * SB;                   // K byte of the float4's first sample
    q_f[q] = f;
    q_lds[q] = r * kMKC + 16 * ((kb >> 4) ^ swz(r)) + (kb & 15);
    src[0][q] = xc + (int64_t)min(I * BT + r, a.n_in - 1) * rsf;
    src[1][q] = xc + (int64_t)min(J * BT + r, a.n_in - 1) * rsf;
  }
  float4 R[PF][NOP][L];
  auto gload = [&](auto S, int st) {
    constexpr int sl = decltype(S)::value;
    const int64_t tb = t0 + (int64_t)st * SPS;
#pragma unroll
    for (int o = 0; o < NOP; ++o)
#pragma unroll
      for (int q = 0; q < L; ++q) {
        const int64_t t = tb + 2 * q_f[q];
        const float* g = src[o][q] + t * 2;
        float4 v;
        if (t + 2 <= t1) {
          v = load16_any<float4>(g);   // rows start 8-byte aligned
        } else {
          v = make_float4(0.f, 0.f, 0.f, 0.f);
          if (t < t1) {
            v.x = g[0];
            v.y = g[1];
          }
        }
        R[sl][o][q] = v;
      }
  };
  auto gload_full = [&](auto S, int st) {   // st < n_full
    constexpr int sl = decltype(S)::value;
    const int64_t tb = t0 + (int64_t)st * SPS;
#pragma unroll
    for (int o = 0; o < NOP; ++o)
#pragma unroll
      for (int q = 0; q < L; ++q) R[sl][o][q] = load16_any<float4>(src[o][q] + (tb + 2 * q_f[q]) * 2);
  };
  auto cvt_store = [&](auto S, int buf) {
    constexpr int sl = decltype(S)::value;
    int8_t* base = lds + buf * STAGE;
#pragma unroll
    for (int o = 0; o < NOP; ++o)
#pragma unroll
      for (int q = 0; q < L; ++q) {
        const float4 v = R[sl][o][q];
        int8_t* d = base + o * PANEL + q_lds[q];
        if constexpr (EKM == kElemF16) {
          *reinterpret_cast<uint2*>(d) = make_uint2(pack_f16x2(v.x, v.y), pack_f16x2(v.z, v.w));
        } else {
          int x = __builtin_amdgcn_cvt_pk_fp8_f32(sc * v.x, sc * v.y, 0, false);
          x = __builtin_amdgcn_cvt_pk_fp8_f32(sc * v.z, sc * v.w, x, true);
          *reinterpret_cast<int*>(d) = x;
        }
      }
  };

  Acc vr[MB][NBN], vi[MB][NBN];
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < NBN; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        vr[m][n][r] = 0;
        vi[m][n][r] = 0;
      }

  const int frow = lane & 31;
  const int g = lane >> 5;
  auto read = [&](int buf, v4i (&af)[MB][2], v4i (&bf)[NBN][2]) {
    const int8_t* As = lds + buf * STAGE;
    const int8_t* Bs = DIAG ? As : As + PANEL;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int cidx = 2 * h + g;
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        const int r = wm * (BT / 2) + m * 32 + frow;
        af[m][h] = *reinterpret_cast<const v4i*>(As + r * kMKC + 16 * (cidx ^ swz(r)));
      }
#pragma unroll
      for (int n = 0; n < NBN; ++n) {
        const int r = (wn * NBN + n) * 32 + frow;
        bf[n][h] = *reinterpret_cast<const v4i*>(Bs + r * kMKC + 16 * (cidx ^ swz(r)));
      }
    }
  };
  // 32 x 32 block (m, n) of this wave: rows MB wm + m, columns wn NBN + n (in
  // blocks); above the diagonal of a diagonal tile it is skipped.
  auto skip = [&](int m, int n) { return DIAG && wn * NBN + n > MB * wm + m; };
  // every block of the wave skipped, or past the last input
  const bool idle = (DIAG && wn * NBN > MB * wm + MB - 1) || I * BT + wm * (BT / 2) >= a.n_in || J * BT + wn * NBN * 32 >= a.n_in;
  auto compute = [&](const v4i (&af)[MB][2], const v4i (&bf)[NBN][2]) {
    v4i ra[MB][2];
    if constexpr (EKM == kElemF8) {
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NBN; ++n)
          if (!skip(m, n)) mfma64<EKM>(af[m], bf[n], vr[m][n]);
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int h = 0; h < 2; ++h) ra[m][h] = rotm4<EKM>(af[m][h]);
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NBN; ++n)
          if (!skip(m, n)) mfma64<EKM>(ra[m], bf[n], vi[m][n]);
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
          for (int n = 0; n < NBN; ++n)
            if (!skip(m, n)) mfma16<EKM>(af[m][h], bf[n][h], vr[m][n]);
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int h = 0; h < 2; ++h) ra[m][h] = rotm4<EKM>(af[m][h]);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
          for (int n = 0; n < NBN; ++n)
            if (!skip(m, n)) mfma16<EKM>(ra[m][h], bf[n][h], vi[m][n]);
    }
  };

  using S0 = std::integral_constant<int, 0>;
  const int n_full = (int)((t1 - t0) / SPS);       // stages whose samples are all there
  const bool deep = DIAG && a.n_tiles == 1 && n_full > PF + 1;
  static_assert(PF == 3 || PF == 4, "the prologue and the unrolled main loop below are written for 3 or 4 slots");
  // prologue: stages 0 .. PF - 1 in flight (slot p holds stage p)
  if (deep) {
    gload_full(S0{}, 0);
    gload_full(std::integral_constant<int, 1>{}, 1);
    gload_full(std::integral_constant<int, 2>{}, 2);
    if constexpr (PF == 4) gload_full(std::integral_constant<int, PF == 4 ? 3 : 0>{}, 3);
    cvt_store(S0{}, 0);
    gload_full(S0{}, PF);
  } else {
    if (0 < n_st) gload(S0{}, 0);
    if (1 < n_st) gload(std::integral_constant<int, 1>{}, 1);
    if (2 < n_st) gload(std::integral_constant<int, 2>{}, 2);
    if constexpr (PF == 4) {
      if (3 < n_st) gload(std::integral_constant<int, PF == 4 ? 3 : 0>{}, 3);
    }
    if (n_st > 0) {
      cvt_store(S0{}, 0);
      if (PF < n_st) gload(S0{}, PF);
    }
  }
  // This wave's LDS accesses are done, then every wave's (loads stay in flight).
  auto barrier = [&] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  __syncthreads();
  // Stage st lives in register slot st % PF; iteration st converts stage
  // st + 1 (freeing its slot) and refills that slot with stage st + 1 + PF.
  auto step = [&](auto full, auto U, int st) {
    constexpr bool FULL = decltype(full)::value;
    constexpr int u = decltype(U)::value;
    constexpr int nx = (u + 1) % PF;
    v4i af[MB][2], bf[NBN][2];
    if (!idle) read(st & 1, af, bf);
    if (FULL || st + 1 < n_st) {
      cvt_store(std::integral_constant<int, nx>{}, (st + 1) & 1);   // the buffer last read in stage st - 1
      if constexpr (FULL) gload_full(std::integral_constant<int, nx>{}, st + 1 + PF);
      else if (st + 1 + PF < n_st) gload(std::integral_constant<int, nx>{}, st + 1 + PF);
    }
    if (!idle) compute(af, bf);
    if constexpr (FULL) barrier();
    else __syncthreads();
  };
  auto steps = [&](auto full, int st) {
    constexpr bool FULL = decltype(full)::value;
    step(full, std::integral_constant<int, 0>{}, st);
    if (FULL || st + 1 < n_st) step(full, std::integral_constant<int, 1>{}, st + 1);
    if (FULL || st + 2 < n_st) step(full, std::integral_constant<int, 2>{}, st + 2);
    if constexpr (PF == 4) {
      if (FULL || st + 3 < n_st) step(full, std::integral_constant<int, PF == 4 ? 3 : 0>{}, st + 3);
    }
  };
  int st0 = 0;
  if (deep)
    for (; st0 + 2 * PF < n_full; st0 += PF) steps(std::true_type{}, st0);
  for (; st0 < n_st; st0 += PF) steps(std::false_type{}, st0);
  if (idle) return;

  // Epilogue (32 x 32 accumulator layout: register r of lane l holds row
  // 8*(r/4) + 4*(l/32) + r%4, column l%32).  FP8 sums are s_c^2 V exactly.
  const float scale = EKM == kElemF8 ? 1.f / (sc * sc) : 1.f;
  const int64_t out0 = (int64_t)split * a.out_split_stride + (int64_t)ch * a.n_products;
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < NBN; ++n) {
      if (skip(m, n)) continue;
      const int j = J * BT + (wn * NBN + n) * 32 + (lane & 31);
#pragma unroll
      for (int h = 0; h < 16; h += 8) {
        uint32_t off[8];
        float2 v[8];
#pragma unroll
        for (int r = h; r < h + 8; ++r) {
          const int i = I * BT + wm * (BT / 2) + m * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          off[r - h] = i < a.n_in && j <= i ? (uint32_t)tri_index(i, j) : kNoProduct;
          v[r - h] = make_float2(vr[m][n][r] * scale, i == j ? 0.f : vi[m][n][r] * scale);
        }
        put_products(static_cast<float2*>(a.out) + out0, off, v, a.accumulate);
      }
    }
}

// int8 variant of mfma_tile_128 on v_mfma_i32_16x16x64_i8: the same staging,
// pipeline and 64 x 64 wave tile, as 4 x 4 blocks of 16 x 16.  Each fragment
// read is one contiguous 1 KB of LDS (16 rows x 64 bytes), and the MFMA moves
// half the accumulator registers per multiply-accumulate of the 32 x 32 x 32
// form; measured on the MI355X it runs the C3 integration ≈4 % faster (the
// clock under load rises from ≈1.67 to ≈1.87 GHz).  A diagonal wave skips the
// 6 strictly upper 16 x 16 blocks of its quarter.
// THROUGH: the products are only stored, through to memory (system scope).
template <int EK, bool DIAG, bool THROUGH = false>
__device__ __forceinline__ void mfma_tile_128_i8(const XArgs& a, int8_t* lds, int ch, int split, int I, int J) {
  constexpr int BT = 128;
  constexpr int PANEL = BT * kMKC;           // bytes per operand per stage
  constexpr int STAGE = PANEL * (DIAG ? 1 : 2);
  constexpr int QPW = BT / 16 / 4;           // 1 KB load instructions per operand per wave
  constexpr int LPW = QPW * (DIAG ? 1 : 2);  // load instructions per wave per stage
  static_assert(EK == kElemI8 || EK == kElemCI4, "16 x 16 x 64 tile is the int8 engine");

  const int8_t* __restrict__ xc = static_cast<const int8_t*>(a.x) + (int64_t)ch * a.ch_stride_b;
  const int64_t k0 = (int64_t)split * a.k_split_bytes;
  const int64_t k1 = min(a.k_bytes, k0 + a.k_split_bytes);
  const int n_st = k1 > k0 ? (int)((k1 - k0 + kMKC - 1) / kMKC) : 0;
  const int64_t last = ((k1 - 1) >> 4) << 4;   // last valid 16-byte chunk start
  // Stages whose 64 bytes all lie in [k0, k1) and whose offsets fit 32 bits.
  const int n_fast = a.row_stride_b < (int64_t(1) << 24) ? (int)((k1 - k0) / kMKC) : 0;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  // This lane's part of each load instruction: LDS row lrow (of 16), chunk p.
  const int lrow = lane >> 2, p = lane & 3;
  const int8_t* gA[QPW];
  const int8_t* gB[QPW];
  uint32_t oA[QPW], oB[QPW];
  int rowq[QPW];
  const int8_t* tA = xc + (int64_t)(I * BT) * a.row_stride_b + k0;
  const int8_t* tB = xc + (int64_t)(J * BT) * a.row_stride_b + k0;
#pragma unroll
  for (int q = 0; q < QPW; ++q) {
    const int r = (wave * QPW + q) * 16 + lrow;    // tile row
    rowq[q] = r;
    const int c = p ^ swz(r);                      // global chunk this lane fetches
    const int ra = min(I * BT + r, a.n_in - 1);
    const int rb = min(J * BT + r, a.n_in - 1);
    gA[q] = xc + (int64_t)ra * a.row_stride_b + 16 * c;
    gB[q] = xc + (int64_t)rb * a.row_stride_b + 16 * c;
    oA[q] = (uint32_t)((int64_t)(ra - I * BT) * a.row_stride_b + 16 * c);
    oB[q] = (uint32_t)((int64_t)(rb - J * BT) * a.row_stride_b + 16 * c);
  }
  auto issue = [&](int st) {
    int8_t* base = lds + (st % kMNS) * STAGE + wave * QPW * 1024;
    if (st < n_fast) {
      const int8_t* ga = tA + st * kMKC;
      const int8_t* gb = tB + st * kMKC;
#pragma unroll
      for (int q = 0; q < QPW; ++q) {
        __builtin_amdgcn_global_load_lds(ga + oA[q], base + q * 1024, 16, 0, 0);
        if (!DIAG) __builtin_amdgcn_global_load_lds(gb + oB[q], base + q * 1024 + PANEL, 16, 0, 0);
      }
    } else {
      const int64_t kb = k0 + (int64_t)st * kMKC;
#pragma unroll
      for (int q = 0; q < QPW; ++q) {
        const int c = p ^ swz(rowq[q]);
        const int64_t kk = kb + 16 * c;
        const int64_t off = (kk <= last ? kb : last - 16 * c);   // keep the 16 bytes inside the row
        __builtin_amdgcn_global_load_lds(gA[q] + off, base + q * 1024, 16, 0, 0);
        if (!DIAG) __builtin_amdgcn_global_load_lds(gB[q] + off, base + q * 1024 + PANEL, 16, 0, 0);
      }
    }
  };
  // Zero / mask the chunks of stage st that reach past k1 (only the last stage).
  auto fix_tail = [&](int st) {
    int8_t* base = lds + (st % kMNS) * STAGE;
    const int64_t kb = k0 + (int64_t)st * kMKC;
#pragma unroll
    for (int q = 0; q < QPW; ++q) {
      const int c = p ^ swz(rowq[q]);
      const int64_t kk = kb + 16 * c;
      if (kk + 16 > k1) {
        const int64_t valid = k1 - kk;
#pragma unroll
        for (int op = 0; op < (DIAG ? 1 : 2); ++op) {
          v4i* cell = reinterpret_cast<v4i*>(base + op * PANEL + (wave * QPW + q) * 1024 + lane * 16);
          v4i v = *cell;
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const int64_t lo = 4 * w;
            const int keep = valid >= lo + 4 ? 4 : (valid > lo ? (int)(valid - lo) : 0);
            const uint32_t m = keep >= 4 ? 0xFFFFFFFFu : ((1u << (8 * keep)) - 1u);
            v[w] = (int)((uint32_t)v[w] & m);
          }
          *cell = v;
        }
      }
    }
  };

  v4i vr[4][4], vi[4][4];
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      vr[m][n] = v4i{0, 0, 0, 0};
      vi[m][n] = v4i{0, 0, 0, 0};
    }

#pragma unroll
  for (int s = 0; s < kMNS - 1; ++s)
    if (s < n_st) issue(s);

  const bool tail = (k1 - k0) % kMKC != 0;
  // Wait for this wave's loads of stage st (later stages stay in flight),
  // mask the K tail, and make stage st visible to all waves.  A plain
  // s_barrier: a fenced one would also drain the later stages' loads.
  auto arrive = [&](int st) {
    const int ahead = min(kMNS - 2, n_st - 1 - st);
    if (ahead >= 2) wait_vmcnt<2 * LPW>();
    else if (ahead == 1) wait_vmcnt<LPW>();
    else wait_vmcnt<0>();
    if (tail && st == n_st - 1) fix_tail(st);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    asm volatile("s_barrier" ::: "memory");
  };
  // 16 x 16 x 64 fragments: lane l reads row (l % 16) of a 16-row block,
  // 16-byte chunk l / 16 (the whole 64-byte stage row across 4 lanes).
  auto read = [&](int st, v4i (&af)[4], v4i (&bf)[4]) {
    const int8_t* As = lds + (st % kMNS) * STAGE;
    const int8_t* Bs = DIAG ? As : As + PANEL;
    const int c = lane >> 4;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int r = wm * 64 + m * 16 + (lane & 15);
      af[m] = *reinterpret_cast<const v4i*>(As + r * kMKC + 16 * (c ^ swz(r)));
    }
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int r = wn * 64 + n * 16 + (lane & 15);
      bf[n] = *reinterpret_cast<const v4i*>(Bs + r * kMKC + 16 * (c ^ swz(r)));
    }
  };
  auto compute = [&](auto sk, const v4i (&af)[4], const v4i (&bf)[4]) {
    constexpr bool SK = decltype(sk)::value;
    if constexpr (EK != kElemCI4) {   // CI4 stages run through compute_ci4
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int n = 0; n < 4; ++n)
          if (!(SK && n > m)) vr[m][n] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[m], bf[n], vr[m][n], 0, 0, 0);
      v4i ra[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) ra[m] = rotm4<kElemI8>(af[m]);
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int n = 0; n < 4; ++n)
          if (!(SK && n > m)) vi[m][n] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ra[m], bf[n], vi[m][n], 0, 0, 0);
    }
  };

  if (n_st > 0) {
    arrive(0);
    if (kMNS - 1 < n_st) issue(kMNS - 1);
  }
  // In a diagonal tile the wave of the strictly upper 64 x 64 quarter only
  // loads its share of the panel and keeps the barriers.
  if (DIAG && wm < wn) {
    for (int s = 0; s + 1 < n_st; ++s) {
      arrive(s + 1);
      if (s + kMNS < n_st) issue(s + kMNS);
    }
    return;
  }
  // CI4: a stage's 16 packed samples per lane feed two K steps (dwords 0-1
  // of every A and B fragment the first, 2-3 the second).  Each step's
  // operands are unpacked just before its 32 MFMAs; once the second step's
  // are unpacked the packed registers take the next stage's LDS reads, which
  // then run under the second step's MFMAs.
  auto unpack_ci4 = [&](int h, const v4i (&pa)[4], const v4i (&pb)[4], v4i (&ua)[4], v4i (&ub)[4]) {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      ua[m] = ci4_plain(pa[m][2 * h], pa[m][2 * h + 1]);
      ub[m] = ci4_plain(pb[m][2 * h], pb[m][2 * h + 1]);
    }
  };
  auto compute_ci4 = [&](auto sk, const v4i (&ua)[4], const v4i (&ub)[4]) {
    constexpr bool SK = decltype(sk)::value;
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int n = 0; n < 4; ++n)
        if (!(SK && n > m)) vr[m][n] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ua[m], ub[n], vr[m][n], 0, 0, 0);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      // -iA = (im, -re): the operand's im words, and its re words negated
      const v4i a = ua[m];
      const v4i ra = {a[1], (int)neg_hi_nibbles((uint32_t)a[0]), a[3], (int)neg_hi_nibbles((uint32_t)a[2])};
#pragma unroll
      for (int n = 0; n < 4; ++n)
        if (!(SK && n > m)) vi[m][n] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ra, ub[n], vi[m][n], 0, 0, 0);
    }
  };
  auto run_ci4 = [&](auto sk) {
    constexpr int NM = (DIAG && decltype(sk)::value) ? 20 : 32;   // MFMAs per K step
    v4i pa[4], pb[4], ua[4], ub[4];
    if (n_st > 0) read(0, pa, pb);
    for (int s = 0; s < n_st; ++s) {
      unpack_ci4(0, pa, pb, ua, ub);
      compute_ci4(sk, ua, ub);
      unpack_ci4(1, pa, pb, ua, ub);
      if (s + 1 < n_st) {
        arrive(s + 1);
        if (s + kMNS < n_st) issue(s + kMNS);
        read(s + 1, pa, pb);
      }
      compute_ci4(sk, ua, ub);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
      }
      __builtin_amdgcn_sched_group_barrier(0x008, NM - 8, 0);
    }
  };
  auto run = [&](auto sk) {
    constexpr int NM = (DIAG && decltype(sk)::value) ? 20 : 32;   // MFMAs per stage
    v4i af0[4], bf0[4], af1[4], bf1[4];
    if (n_st > 0) read(0, af0, bf0);
    for (int s = 0; s + 1 < n_st; ++s) {
      arrive(s + 1);
      if (s + kMNS < n_st) issue(s + kMNS);
      read(s + 1, af1, bf1);
      compute(sk, af0, bf0);
#pragma unroll
      for (int q = 0; q < (NM < 8 ? NM : 8); ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
      }
      if constexpr (NM > 8) __builtin_amdgcn_sched_group_barrier(0x008, NM - 8, 0);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        af0[m] = af1[m];
        bf0[m] = bf1[m];
      }
    }
    if (n_st > 0) compute(sk, af0, bf0);
  };
  if constexpr (EK == kElemCI4) {
    if (DIAG && wm == wn) run_ci4(std::true_type{});
    else run_ci4(std::false_type{});
  } else {
    if (DIAG && wm == wn) run(std::true_type{});
    else run(std::false_type{});
  }

  // Epilogue.  16 x 16 accumulator layout: register r of lane l holds row
  // 4*(l/16) + r, column l%16.
  // A later pass of the integration, eight products at a time.
  if constexpr (!THROUGH) if (a.accumulate) {
    int2* const sum = static_cast<int2*>(a.out) + (int64_t)split * a.out_split_stride + (int64_t)ch * a.n_products;
#pragma unroll
    for (int mn = 0; mn < 16; mn += 2) {
      int lq = lane;
      asm volatile("" : "+v"(lq));   // indexes made here, not all at once ahead of the loop over K
      uint32_t off[8];
      int2 v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int m = (mn + q / 4) / 4, n = (mn + q / 4) % 4;
        const int i = I * BT + wm * 64 + m * 16 + 4 * (lq >> 4) + q % 4;
        const int j = J * BT + wn * 64 + n * 16 + (lq & 15);
        off[q] = i < a.n_in && j <= i ? (uint32_t)tri_index(i, j) : kNoProduct;
        v[q] = make_int2(EK == kElemCI4 ? vr[m][n][q % 4] >> 8 : vr[m][n][q % 4], i == j ? 0 : EK == kElemCI4 ? vi[m][n][q % 4] >> 8 : vi[m][n][q % 4]);
      }
      add_products(sum, off, v);
    }
    return;
  }
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int j = J * BT + wn * 64 + n * 16 + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = I * BT + wm * 64 + m * 16 + 4 * (lane >> 4) + r;
        if (i < a.n_in && j <= i) {
          const int64_t off = (int64_t)split * a.out_split_stride + (int64_t)ch * a.n_products + tri_index(i, j);
          int2* pp = static_cast<int2*>(a.out) + off;
          // CI4 operands are 16 x the sample parts: the sums are 256 V exactly
          const int re = EK == kElemCI4 ? (vr[m][n][r] >> 8) : vr[m][n][r];
          const int im = (i == j) ? 0 : (EK == kElemCI4 ? (vi[m][n][r] >> 8) : vi[m][n][r]);
          if constexpr (THROUGH) {
            __hip_atomic_store(reinterpret_cast<uint64_t*>(pp), (uint64_t)(uint32_t)re | (uint64_t)(uint32_t)im << 32,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
          } else {
            *pp = make_int2(re, im);
          }
        }
      }
    }
}

template <int EK>
__global__ __launch_bounds__(256, 2) void xeng_mfma_128_kernel(XArgs a) {
  __shared__ __attribute__((aligned(1024))) int8_t lds[kMNS * 2 * 128 * kMKC];
  const int64_t slot = blockIdx.x / kNumXcd;
  const int64_t item = xcd_item(blockIdx.x, a.per_xcd);
  if (slot >= a.per_xcd || item >= a.n_items) return;
  int ch, split, I, J;
  item_decode(a, item, ch, split, I, J);
  if constexpr (EK == kElemI8 || EK == kElemCI4) {
    if (I == J) mfma_tile_128_i8<EK, true>(a, lds, ch, split, I, J);
    else mfma_tile_128_i8<EK, false>(a, lds, ch, split, I, J);
  } else {
    if (I == J) mfma_tile_128<EK, true>(a, lds, ch, split, I, J);
    else mfma_tile_128<EK, false>(a, lds, ch, split, I, J);
  }
}

// The converting FP16 engine on 129 to 256 inputs, one workgroup per channel: 8 waves
// cover the 36 blocks of 32 x 32 on or below the diagonal, so that every float32
// row is read once, where three 128-row tiles read each twice and find the second
// reading in L2 only while they keep step (4.9 GB read for 4.3 of samples at 256
// x 512 x 4096; 8.1 with loads that do not wait for each other).  256 x 512 x 4096
// with its read-out 1276 -> 940 us, 130 x 512 x 2000 554 -> 374, 200 x 256 x 2000 346 ->
// 264.  Bound by the loads of float32 samples (5 TB/s).
//
// Block rows come in pairs (7 - p, p) of 9 blocks; waves p and p + 4 (one SIMD)
// take 5 and 4 of them: 160 accumulators, and two stages of samples in flight (4
// float4 per thread and stage).  A wave reads both operands of every block from
// LDS; a wave of 4 repeats its last one, because a branch around a block made the
// compiler spill 215 registers.  Samples past
// the pass are zero; rows past N_I are read from a clamped row and never stored.
__device__ __forceinline__ void mfma_tri_cvt(const XArgs& a, int8_t* lds, int ch, int split) {
  constexpr int BT = 256, NT = 512;
  constexpr int STAGE = BT * kMKC;
  constexpr int SPS = kMKC / 4, NF = SPS / 2;     // samples, float4 per row and stage
  constexpr int L = BT * NF / NT;                 // float4 per thread and stage
  constexpr int PF = 2;                           // stages in flight in registers
  constexpr int NB = 5;                           // blocks per wave, at most

  const float* __restrict__ xc = reinterpret_cast<const float*>(static_cast<const int8_t*>(a.x) + (int64_t)ch * a.ch_stride_b);
  const int64_t k0 = (int64_t)split * a.k_split_bytes;
  const int64_t k1 = min(a.k_bytes, k0 + a.k_split_bytes);
  const int n_st = k1 > k0 ? (int)((k1 - k0 + kMKC - 1) / kMKC) : 0;
  const int64_t t0 = k0 / 4, t1 = k1 / 4;          // sample range of the pass
  const int n_full = (int)((t1 - t0) / SPS);       // stages whose samples are all there
  const int64_t rsf = a.row_stride_b / 4;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // This thread's loads: float4 f of rows tid / NF + 64 q.
  const int f = tid % NF;
  uint32_t src[L];   // 32 bits suffice: the caller has checked the stride
#pragma unroll
  for (int q = 0; q < L; ++q) src[q] = (uint32_t)min(tid / NF + NT / NF * q, a.n_in - 1) * (uint32_t)rsf + 4 * f;
  // (64 rows on, the swizzle is the same)
  const int q_lds = (tid / NF) * kMKC + 16 * ((f >> 1) ^ swz(tid / NF)) + 8 * (f & 1);
  float4 R[PF][L];
  auto gload_full = [&](auto S, int st) {   // st < n_full
    constexpr int sl = decltype(S)::value;
    const float* base = xc + (t0 + (int64_t)st * SPS) * 2;
#pragma unroll
    for (int q = 0; q < L; ++q) R[sl][q] = load16_any<float4>(base + src[q]);
  };
  auto gload = [&](auto S, int st) {
    constexpr int sl = decltype(S)::value;
    const int64_t t = t0 + (int64_t)st * SPS + 2 * f;
#pragma unroll
    for (int q = 0; q < L; ++q) {
      const float* g = xc + (t0 + (int64_t)st * SPS) * 2 + src[q];
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (t + 2 <= t1) {
        v = load16_any<float4>(g);
      } else if (t < t1) {
        v.x = g[0];
        v.y = g[1];
      }
      R[sl][q] = v;
    }
  };
  auto cvt_store = [&](auto S, int buf) {
    constexpr int sl = decltype(S)::value;
#pragma unroll
    for (int q = 0; q < L; ++q) {
      const float4 v = R[sl][q];
      *reinterpret_cast<uint2*>(lds + buf * STAGE + q_lds + NT / NF * kMKC * q) = make_uint2(pack_f16x2(v.x, v.y), pack_f16x2(v.z, v.w));
    }
  };

  // This wave's blocks (not stored where they are a repetition or past the last input).
  const int p = wave & 3, q0 = wave < 4 ? 0 : 5;
  int br[NB], bc[NB];
  bool on[NB];
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    const int q = min(q0 + k, 8);
    br[k] = q < 8 - p ? 7 - p : p;
    bc[k] = q < 8 - p ? q : q - (8 - p);
    on[k] = q0 + k <= 8 && br[k] * 32 < a.n_in;
  }
  v16f vr[NB], vi[NB];
#pragma unroll
  for (int k = 0; k < NB; ++k)
#pragma unroll
    for (int r = 0; r < 16; ++r) vr[k][r] = vi[k][r] = 0.f;

  const int frow = lane & 31, g = lane >> 5;
  const int fr[2] = {frow * kMKC + 16 * (g ^ swz(frow)), frow * kMKC + 16 * ((2 + g) ^ swz(frow))};
  auto compute = [&](int buf) {
    const int8_t* S = lds + buf * STAGE;
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      v4i af[2], bf[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        af[h] = *reinterpret_cast<const v4i*>(S + br[k] * 32 * kMKC + fr[h]);
        bf[h] = *reinterpret_cast<const v4i*>(S + bc[k] * 32 * kMKC + fr[h]);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) mfma16<kElemF16>(af[h], bf[h], vr[k]);
#pragma unroll
      for (int h = 0; h < 2; ++h) mfma16<kElemF16>(rotm4<kElemF16>(af[h]), bf[h], vi[k]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // This wave's LDS accesses are done, then every wave's (loads stay in flight).
  auto barrier = [&] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  const bool deep = n_full > PF + 1;
  if (deep) {
    gload_full(S0{}, 0);
    gload_full(S1{}, 1);
    cvt_store(S0{}, 0);
    gload_full(S0{}, 2);
  } else {
    if (0 < n_st) gload(S0{}, 0);
    if (1 < n_st) gload(S1{}, 1);
    if (0 < n_st) cvt_store(S0{}, 0);
    if (2 < n_st) gload(S0{}, 2);
  }
  barrier();
  // Stage st lives in register slot st % PF; iteration st converts stage st + 1
  // (freeing its slot), refills that slot with stage st + 1 + PF and multiplies
  // stage st.  FULL: these exist and are whole, so that no condition stands around
  // the loads and the compiler waits for the oldest stage only.
  auto step = [&](auto full, auto NX, int st) {
    constexpr bool FULL = decltype(full)::value;
    if (FULL || st + 1 < n_st) {
      cvt_store(NX, (st + 1) & 1);
      if constexpr (FULL) gload_full(NX, st + 1 + PF);
      else if (st + 1 + PF < n_st) gload(NX, st + 1 + PF);
    }
    compute(st & 1);
    barrier();
  };
  int st = 0;
  if (deep)
    for (; st + 2 + PF < n_full; st += 2) {
      step(std::true_type{}, S1{}, st);
      step(std::true_type{}, S0{}, st + 1);
    }
  for (; st < n_st; st += 2) {
    step(std::false_type{}, S1{}, st);
    if (st + 1 < n_st) step(std::false_type{}, S0{}, st + 1);
  }

  // Epilogue (32 x 32 accumulator layout: register r of lane l holds row
  // 8*(r/4) + 4*(l/32) + r%4, column l%32).
  float2* const out = static_cast<float2*>(a.out) + (int64_t)split * a.out_split_stride + (int64_t)ch * a.n_products;
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    const int j = bc[k] * 32 + (lane & 31);
#pragma unroll
    for (int h = 0; h < 16; h += 8) {
      uint32_t off[8];
      float2 v[8];
#pragma unroll
      for (int r = h; r < h + 8; ++r) {
        const int i = br[k] * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        off[r - h] = on[k] && i < a.n_in && j <= i ? (uint32_t)tri_index(i, j) : kNoProduct;
        v[r - h] = make_float2(vr[k][r], i == j ? 0.f : vi[k][r]);
      }
      put_products(out, off, v, a.accumulate);
    }
  }
}

__global__ __launch_bounds__(512, 1) void xeng_cvt_tri_kernel(XArgs a) {
  __shared__ __attribute__((aligned(1024))) int8_t lds[2 * 256 * kMKC];
  const int64_t slot = blockIdx.x / kNumXcd;
  const int64_t item = xcd_item(blockIdx.x, a.per_xcd);
  if (slot >= a.per_xcd || item >= a.n_items) return;
  mfma_tri_cvt(a, lds, (int)(item / a.n_split), (int)(item % a.n_split));
}

// Waves per workgroup of the converting engines (one workgroup per CU).  FP16:
// 8 (two per SIMD, 64 x 32 wave parts, 177 VGPRs), 8 % faster on C4 than 4
// waves of 64 x 64.  FP8 stages twice the samples per row and would spill
// with 8, so it keeps 4 (measured slower with 8).
template <int EK>
constexpr int cvt_waves() { return EK == kElemF16Cvt ? 8 : 4; }

template <int EK>
__global__ __launch_bounds__(cvt_waves<EK>() * 64, 1) void xeng_cvt_128_kernel(XArgs a) {
  __shared__ __attribute__((aligned(1024))) int8_t lds[2 * 2 * 128 * kMKC];
  const int64_t slot = blockIdx.x / kNumXcd;
  const int64_t item = xcd_item(blockIdx.x, a.per_xcd);
  if (slot >= a.per_xcd || item >= a.n_items) return;
  int ch, split, I, J;
  item_decode(a, item, ch, split, I, J);
  if (I == J) mfma_tile_cvt<EK, 128, true, cvt_waves<EK>()>(a, lds, ch, split, I, J);
  else mfma_tile_cvt<EK, 128, false, cvt_waves<EK>()>(a, lds, ch, split, I, J);
}

// Up to 64 inputs: one 64-row tile per channel.
template <int EK>
__global__ __launch_bounds__(256, EK == kElemF16Cvt ? 4 : 3) void xeng_cvt_64_kernel(XArgs a) {
  __shared__ __attribute__((aligned(1024))) int8_t lds[2 * 64 * kMKC];
  const int64_t slot = blockIdx.x / kNumXcd;
  const int64_t item = xcd_item(blockIdx.x, a.per_xcd);
  if (slot >= a.per_xcd || item >= a.n_items) return;
  int ch, split, I, J;
  item_decode(a, item, ch, split, I, J);
  mfma_tile_cvt<EK, 64, true, 4>(a, lds, ch, split, I, J);
}

// FP32 matrix-core tile: the 64-row tile of mfma_tile (same staging,
// pipeline and swizzle), but each wave's 32 x 32 quadrant runs as 2 x 2
// blocks of v_mfma_f32_16x16x4_f32.  A lane reads one 16-byte chunk (two
// complex samples) of its block row per stage -- row lane % 16, chunk lane /
// 16 -- and instruction q takes float q of it from A and from B, so the 16
// K elements of the stage enter once each, in the same place for both.  In a
// diagonal tile the quadrant waves skip their strictly upper 16 x 16 block:
// 2560 products computed per 2080 needed at 64 inputs, against 3072 with
// 32 x 32 blocks.
typedef float v4f __attribute__((ext_vector_type(4)));

template <bool DIAG>
__device__ __forceinline__ void mfma_tile_f32(const XArgs& a, int8_t* lds, int ch, int split, int I, int J) {
  constexpr int BT = 64;
  constexpr int PANEL = BT * kMKC;
  constexpr int STAGE = PANEL * (DIAG ? 1 : 2);
  constexpr int QPW = BT / 16 / 4;
  constexpr int LPW = QPW * (DIAG ? 1 : 2);

  const int8_t* __restrict__ xc = static_cast<const int8_t*>(a.x) + (int64_t)ch * a.ch_stride_b;
  const int64_t k0 = (int64_t)split * a.k_split_bytes;
  const int64_t k1 = min(a.k_bytes, k0 + a.k_split_bytes);
  const int n_st = k1 > k0 ? (int)((k1 - k0 + kMKC - 1) / kMKC) : 0;
  const int64_t last = ((k1 - 1) >> 4) << 4;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const bool wave_idle = DIAG && (wm < wn);
  const bool quad_diag = DIAG && (wm == wn);

  const int lrow = lane >> 2, p = lane & 3;
  const int8_t* gA[QPW];
  const int8_t* gB[QPW];
  int rowq[QPW];
#pragma unroll
  for (int q = 0; q < QPW; ++q) {
    const int r = (wave * QPW + q) * 16 + lrow;
    rowq[q] = r;
    const int c = p ^ swz(r);
    gA[q] = xc + (int64_t)min(I * BT + r, a.n_in - 1) * a.row_stride_b + 16 * c;
    if (!DIAG) gB[q] = xc + (int64_t)min(J * BT + r, a.n_in - 1) * a.row_stride_b + 16 * c;
  }
  auto issue = [&](int st) {
    int8_t* base = lds + (st % kMNS) * STAGE;
    const int64_t kb = k0 + (int64_t)st * kMKC;
#pragma unroll
    for (int q = 0; q < QPW; ++q) {
      const int c = p ^ swz(rowq[q]);
      const int64_t kk = kb + 16 * c;
      const int64_t off = (kk <= last ? kb : last - 16 * c);
      int8_t* dst = base + (wave * QPW + q) * 1024;
      __builtin_amdgcn_global_load_lds(gA[q] + off, dst, 16, 0, 0);
      if (!DIAG) __builtin_amdgcn_global_load_lds(gB[q] + off, dst + PANEL, 16, 0, 0);
    }
  };
  auto fix_tail = [&](int st) {
    int8_t* base = lds + (st % kMNS) * STAGE;
    const int64_t kb = k0 + (int64_t)st * kMKC;
#pragma unroll
    for (int q = 0; q < QPW; ++q) {
      const int c = p ^ swz(rowq[q]);
      const int64_t kk = kb + 16 * c;
      if (kk + 16 > k1) {
        const int64_t valid = k1 - kk;
#pragma unroll
        for (int op = 0; op < (DIAG ? 1 : 2); ++op) {
          v4i* cell = reinterpret_cast<v4i*>(base + op * PANEL + (wave * QPW + q) * 1024 + lane * 16);
          v4i v = *cell;
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const int64_t lo = 4 * w;
            const int keep = valid >= lo + 4 ? 4 : (valid > lo ? (int)(valid - lo) : 0);
            const uint32_t m = keep >= 4 ? 0xFFFFFFFFu : ((1u << (8 * keep)) - 1u);
            v[w] = (int)((uint32_t)v[w] & m);
          }
          *cell = v;
        }
      }
    }
  };

  v4f vr[2][2], vi[2][2];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      vr[m][n] = v4f{0.f, 0.f, 0.f, 0.f};
      vi[m][n] = v4f{0.f, 0.f, 0.f, 0.f};
    }

#pragma unroll
  for (int s = 0; s < kMNS - 1; ++s)
    if (s < n_st) issue(s);

  const int frow = lane & 15;
  const int c4 = lane >> 4;
  const bool tail = (k1 - k0) % kMKC != 0;
  for (int s = 0; s < n_st; ++s) {
    const int ahead = min(kMNS - 2, n_st - 1 - s);
    if (ahead >= 2) wait_vmcnt<2 * LPW>();
    else if (ahead == 1) wait_vmcnt<LPW>();
    else wait_vmcnt<0>();
    if (tail && s == n_st - 1) {
      fix_tail(s);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    asm volatile("s_barrier" ::: "memory");
    if (s + kMNS - 1 < n_st) issue(s + kMNS - 1);
    if (!wave_idle) {
      const int8_t* As = lds + (s % kMNS) * STAGE;
      const int8_t* Bs = DIAG ? As : As + PANEL;
      v4i af[2], bf[2], bj[2];
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const int r = wm * 32 + m * 16 + frow;
        af[m] = *reinterpret_cast<const v4i*>(As + r * kMKC + 16 * (c4 ^ swz(r)));
      }
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const int r = wn * 32 + n * 16 + frow;
        bf[n] = *reinterpret_cast<const v4i*>(Bs + r * kMKC + 16 * (c4 ^ swz(r)));
        bj[n] = rot4<kElemF32>(bf[n]);
      }
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          if (quad_diag && m < n) continue;   // strictly upper 16 x 16 block
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            vr[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(__int_as_float(af[m][q]), __int_as_float(bf[n][q]),
                                                            vr[m][n], 0, 0, 0);
            vi[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(__int_as_float(af[m][q]), __int_as_float(bj[n][q]),
                                                            vi[m][n], 0, 0, 0);
          }
        }
    }
  }

  if (wave_idle) return;
  // Epilogue.  16 x 16 accumulator layout: register r of lane l holds row
  // 4*(l/16) + r, column l%16.
  const int64_t out0 = (int64_t)split * a.out_split_stride + (int64_t)ch * a.n_products;
  // (rows past the last input are passed by, as in mfma_tile: 1 x 162 x 31 6.24 ->
  // 5.64 us, 14 x 12 x 1117 13.84 -> 13.32)
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    const int i0 = I * BT + __builtin_amdgcn_readfirstlane(wm) * 32 + m * 16;
    if (i0 >= a.n_in) break;                   // rows past the last input
    const TriRow row(i0 + 4 * (lane >> 4));
    uint32_t off[8];
    float2 v[8];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const int j = J * BT + wn * 32 + n * 16 + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = (int)row.i + r;
        off[4 * n + r] = !(quad_diag && m < n) && i < a.n_in && j <= i ? row.at(r) + (uint32_t)j : kNoProduct;
        v[4 * n + r] = make_float2(vr[m][n][r], i == j ? 0.f : vi[m][n][r]);
      }
    }
    put_products(static_cast<float2*>(a.out) + out0, off, v, a.accumulate);
  }
}

// Diagonal or off-diagonal tile of the BT-row engine (one instantiation site
// for every kernel that runs BT-row tiles).
template <int EK, int BT>
__device__ __forceinline__ void mfma_tile_any(const XArgs& a, int8_t* lds, int ch, int split, int I, int J) {
  if constexpr (EK == kElemF32) {
    static_assert(BT == 64, "the FP32 matrix-core engine runs 64-row tiles");
    if (I == J) mfma_tile_f32<true>(a, lds, ch, split, I, J);
    else mfma_tile_f32<false>(a, lds, ch, split, I, J);
  } else {
    if (I == J) mfma_tile<EK, BT, true>(a, lds, ch, split, I, J);
    else mfma_tile<EK, BT, false>(a, lds, ch, split, I, J);
  }
}

template <int EK, int BT>
__global__ __launch_bounds__(256, 2) void xeng_mfma_kernel(XArgs a) {
  __shared__ __attribute__((aligned(1024))) int8_t lds[kMNS * 2 * BT * kMKC];
  const int64_t slot = blockIdx.x / kNumXcd;
  const int64_t item = xcd_item(blockIdx.x, a.per_xcd);
  if (slot >= a.per_xcd || item >= a.n_items) return;
  int ch, split, I, J;
  item_decode(a, item, ch, split, I, J);
  mfma_tile_any<EK, BT>(a, lds, ch, split, I, J);
}

// Serving: a device queue of integration jobs shared by persistent grids.
// The host scheduler publishes each admitted job in a slot (its sample and
// output pointers and shape) and lists the slots whose jobs have unclaimed
// items; every workgroup of the running serving grid claims work items --
// (channel, 128-row tile) pairs -- from the listed jobs in turn (round robin
// over the jobs: a small job is not queued behind a large one, and the claims
// of the grid's workgroups spread over the jobs' counters), runs the tile
// over all of the job's samples, and counts it done.  The workgroup that claims a job's last item reports it to
// the host (which then lists the job no more); the workgroup that finishes
// the job's last item writes the job's completion word in host memory.
//
// A claim is one fetch-and-add on the slot's claim word.  It cannot fail, only
// overshoot (a count past the job's items, harmless: the next job of the slot
// sets the word anew), so the few hundred workgroups that meet on one new job
// take its items in as many atomics.  With a compare-and-swap bounded by a
// claim limit all but one of them failed each time: 12 jobs of 64 or 256
// channels and 16 to 128 inputs took 940 us as a batch
// (with one update launch for three copies a job), 700 with the add, and 460
// once a tile's products went through to memory instead of a release fence per
// tile (1500 at first).  serve_claim (serve_queue.h) says why a claim made
// from an entry of an old list is sound.
//
// A grid ends as a whole: once no workgroup has claimed an item for
// idle_ticks of the 100 MHz wall clock, the first workgroup to notice closes
// the grid (it raises `closing` to the grid's generation and tells the host),
// and from then on no workgroup of that generation claims again; each exits
// after its current tile.  So a running grid never thins out to a few
// workgroups that would then carry new work alone; work published after the
// close waits for the next grid, which the scheduler launches at full size.
__device__ __forceinline__ uint64_t sys_load64(const void* p) {
  return __hip_atomic_load(static_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The queue's memory as the kernels reach it: loads and stores of system scope
// go past the caches, and every value is there before what depends on it is
// issued.
struct ServeMemory {
  __device__ uint64_t load(const uint64_t* p) { return sys_load64(p); }
  __device__ uint32_t load_agent(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // two loads in flight together
  __device__ void load2(const uint64_t* p0, const uint64_t* p1, uint64_t& v0, uint64_t& v1) {
    v0 = load(p0);
    v1 = load(p1);
  }
  // *claim += 1 (w: its former value) and a load, in flight together
  __device__ void add_load(uint64_t* claim, const uint64_t* p, uint64_t& w, uint64_t& v) {
    w = __hip_atomic_fetch_add(claim, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    v = load(p);
  }
  __device__ void store(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  template <typename T>
  __device__ void exchange(T* p, T v) {
    __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ void settle() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  }
  // An item was claimed: the grid is busy.
  __device__ void claimed(const ServeQueue& q) {
    __hip_atomic_fetch_max(q.last_claim, (uint64_t)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // Nothing to claim: true once the grid has closed, which the first workgroup
  // to see the queue idle for idle_ticks does; else wait a little.
  __device__ bool idle(const ServeQueue& q) {
    const uint64_t last = __hip_atomic_load(q.last_claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((uint64_t)wall_clock64() > last + q.idle_ticks) {
      uint32_t c = load_agent(q.closing);
      while (c < q.gen && !__hip_atomic_compare_exchange_strong(q.closing, &c, q.gen, __ATOMIC_RELAXED,
                                                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
      }
      if (c < q.gen) __hip_atomic_store(q.host_closing, q.gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      return true;
    }
    __builtin_amdgcn_s_sleep(8);
    return false;
  }
};

// The job's arguments and the claimed item pass through the start of the
// tile's LDS buffer (one LDS object per kernel: a second one makes the
// compiler wait for every LDS-bound global load before each LDS read).
struct ServeClaim {
  ServeJob job;
  int32_t slot, item;
};

__global__ __launch_bounds__(256, 2) void xeng_serve_kernel(ServeQueue q) {
  __shared__ __attribute__((aligned(1024))) int8_t lds[kMNS * 2 * 128 * kMKC];
  static_assert(sizeof(ServeClaim) <= sizeof(lds), "claim record fits in the tile buffer");
  constexpr int kWords = sizeof(ServeJob) / 8;
  static_assert(sizeof(ServeJob) % 8 == 0 && kWords <= 64, "one lane a word");
  ServeClaim* sc = reinterpret_cast<ServeClaim*>(lds);
  if (threadIdx.x == 0)   // a new grid counts as activity: it lingers idle_ticks before it may close
    __hip_atomic_fetch_max(q.last_claim, (uint64_t)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  ServeMemory mem;
  ServeView view{blockIdx.x, 1, 0, 0, 0, true, false};
  for (;;) {
    __syncthreads();   // the previous tile's LDS reads are done
    if (threadIdx.x < 64) {
      int slot = -1;
      uint64_t word = 0;
      if (threadIdx.x == 0) slot = serve_claim(mem, q, view, &word);
      slot = __builtin_amdgcn_readfirstlane(slot);
      if (slot >= 0 && __builtin_amdgcn_readfirstlane((int)view.acquire)) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");
      if (slot >= 0 && threadIdx.x < kWords)
        reinterpret_cast<uint64_t*>(&sc->job)[threadIdx.x] =
            sys_load64(reinterpret_cast<const uint64_t*>(q.slots + slot) + threadIdx.x);
      if (threadIdx.x == 0) {
        sc->item = (int)(uint32_t)word;
        sc->slot = slot;
      }
    }
    __syncthreads();
    const int slot = __builtin_amdgcn_readfirstlane(sc->slot);
    if (slot < 0) return;
    // the record in scalar registers, as a kernel argument would be
    ServeJob job;
#pragma unroll
    for (int k = 0; k < 2 * kWords; ++k)
      reinterpret_cast<int*>(&job)[k] = __builtin_amdgcn_readfirstlane(reinterpret_cast<const int*>(&sc->job)[k]);
    const XArgs& a = job.x;
    const int item = __builtin_amdgcn_readfirstlane(sc->item);
    __syncthreads();   // everyone holds the claim before the tile reuses the buffer
    const int tile = item % a.n_tiles;
    const int ch = item / a.n_tiles;
    int I, J;
    tile_decode(tile, I, J);
    if (I == J) mfma_tile_128_i8<kElemI8, true, true>(a, lds, ch, 0, I, J);
    else mfma_tile_128_i8<kElemI8, false, true>(a, lds, ch, 0, I, J);
    // The products were stored through to memory (system scope), so they are
    // visible device-wide once each wave's stores are acknowledged; a release
    // fence per tile would write back the whole L2 of the XCD.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
      const uint32_t old = __hip_atomic_fetch_add(q.done + (size_t)slot * kServeLine, 1u, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
      if (old + 1 == (uint32_t)a.n_items) {
        __threadfence_system();
        __hip_atomic_store(job.flag, job.flag_value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
      }
    }
  }
}

// Publish a batch of admitted jobs to the queue of a running serving grid
// (serve_publish).  Every store goes through to memory (system scope, or an
// atomic) and is acknowledged before the next step, so no fence has to write
// back an L2.  One launch a batch: as three copies a job the queue updates took
// 8 us each on the device and 25 us a job on the host.
__global__ __launch_bounds__(256) void xeng_publish_kernel(const ServeUpdate* __restrict__ u, int n_jobs, int n_active,
                                                           uint32_t version, ServeQueue q) {
  static_assert(kServeSlots < 256, "a thread per slot, and one for the list's head");
  ServeMemory mem;
  serve_publish(mem, u, n_jobs, n_active, version, q, (int)threadIdx.x, 256);
}

// The launch's own status, here and in launch_xeng_serve: hipGetLastError may
// give an error that a job's fill left behind in the scheduler's thread, and an
// update that was queued must not be taken for one that was not (its jobs would
// be failed, and their slots and arena regions given away, with the update still
// to come).
hipError_t launch_xeng_publish(const ServeUpdate* u, int n_jobs, int n_active, uint32_t version, const ServeQueue& q,
                               hipStream_t s) {
  if (n_jobs > kServeSlots || n_active > kServeSlots) return hipErrorInvalidValue;
  ServeQueue queue = q;
  void* args[] = {&u, &n_jobs, &n_active, &version, &queue};
  return hipLaunchKernel(reinterpret_cast<const void*>(&xeng_publish_kernel), dim3(1), dim3(256), args, 0, s);
}

hipError_t launch_xeng_mfma(const XArgs& a, int elem, int bt, hipStream_t s) {
  const int64_t grid = (int64_t)a.per_xcd * kNumXcd;
  if (grid <= 0) return hipSuccess;
  const dim3 g((unsigned)grid), b(256);
#define CORR_LAUNCH(EK, BT) hipLaunchKernelGGL((xeng_mfma_kernel<EK, BT>), g, b, 0, s, a)
#define CORR_LAUNCH_W2(EK) hipLaunchKernelGGL((xeng_mfma_128_kernel<EK>), g, b, 0, s, a)
  if (elem == kElemI8) {
    if (bt == 128) CORR_LAUNCH_W2(kElemI8); else CORR_LAUNCH(kElemI8, 64);
  } else if (elem == kElemF32) {
    CORR_LAUNCH(kElemF32, 64);   // 64-row tiles only
  } else if (elem == kElemCI4) {
    if (bt == 128) CORR_LAUNCH_W2(kElemCI4); else CORR_LAUNCH(kElemCI4, 64);
  } else if (elem == kElemF16Cvt && bt == 64) {
    hipLaunchKernelGGL((xeng_cvt_64_kernel<kElemF16Cvt>), g, b, 0, s, a);
  } else if (elem == kElemF8Cvt && bt == 64) {
    hipLaunchKernelGGL((xeng_cvt_64_kernel<kElemF8Cvt>), g, b, 0, s, a);
  } else if (elem == kElemF16Cvt && bt == 256) {
    hipLaunchKernelGGL(xeng_cvt_tri_kernel, g, dim3(512), 0, s, a);
  } else if (elem == kElemF16Cvt) {
    hipLaunchKernelGGL((xeng_cvt_128_kernel<kElemF16Cvt>), g, dim3(cvt_waves<kElemF16Cvt>() * 64), 0, s, a);
  } else if (elem == kElemF8Cvt) {
    hipLaunchKernelGGL((xeng_cvt_128_kernel<kElemF8Cvt>), g, dim3(cvt_waves<kElemF8Cvt>() * 64), 0, s, a);
  } else if (elem == kElemF16) {
    if (bt == 128) CORR_LAUNCH_W2(kElemF16); else CORR_LAUNCH(kElemF16, 64);
  } else {
    if (bt == 128) CORR_LAUNCH_W2(kElemF8); else CORR_LAUNCH(kElemF8, 64);
  }
#undef CORR_LAUNCH
#undef CORR_LAUNCH_W2
  return hipGetLastError();
}

hipError_t launch_xeng_serve(const ServeQueue& q, int grid, hipStream_t s) {
  if (grid <= 0) return hipSuccess;
  ServeQueue queue = q;
  void* args[] = {&queue};
  return hipLaunchKernel(reinterpret_cast<const void*>(&xeng_serve_kernel), dim3((unsigned)grid), dim3(256), args, 0, s);
}

int serve_blocks_per_cu() {
  int n = 0;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, xeng_serve_kernel, 256, 0) == hipSuccess ? n : 0;
}

}  // namespace corr
