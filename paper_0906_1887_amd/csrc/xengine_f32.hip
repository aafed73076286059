// Plain FP32 X-engine: V_ij[c] += sum_t x_i[c,t] conj(x_j[c,t]) with FP32
// vector FMAs and FP32 accumulation, for complex float32 or complex int8
// samples (int8 converted exactly to float when staged), rows of any sample
// alignment.
//
// The cross-multiply-accumulate of Sec. 4 ("third step") on the vector ALUs,
// the precision the paper used throughout.  The paper's fastest design shares
// each input sample among a small group of products through shared memory
// (group parallel, G = 4).  Here a workgroup of 16 x 16 threads stages 16
// samples of two panels of BT = 64 inputs in LDS, and each thread keeps an R x
// R block (R = 4) of complex accumulators in registers, so every LDS read feeds
// R complex MACs.
//
// Work items.  Off-diagonal tile: the panels are the rows of I and of J, thread
// (ty, tx) forms rows ty against columns tx.  Diagonal tiles come in pairs (of
// one channel or of neighbouring channels): the panels are the rows of the
// two tiles, and two waves take each tile, a thread one of its 120 strictly
// lower blocks or of its first 8 diagonal ones; the other 8 diagonal blocks of
// both are dealt out R R / 16 products a thread.  (A square diagonal tile, as
// before, computes every product twice.)
//
// Up to 32 inputs: a panel holds two channels' 32 rows, or four channels' 16, so
// that a workgroup takes 4 or 8 channels, each with 36 or 10 lanes of one wave (a
// block each).  In pairs of 64-row tiles most blocks lay past the last input: 21
// inputs x 652 channels x 2771 samples 378 -> 199 us a pass, 32 x 128 x 1000 48 ->
// 37, 16 x 734 x 1000 173 -> 59, 4 x 600 x 5000 538 -> 164, 32 x 600 x 2000 int8 224
// -> 127.
//
// Bound: FP32 vector rate: four items a CU run at 100 TFLOP/s of executed FMAs
// (115 VGPRs, four waves per SIMD).  With square diagonal tiles of 128 rows
// and two waves per SIMD before: 128 inputs x 96 channels x 2000 samples 343
// -> 201 us a pass, 64 x 128 x 1000 86 -> 54 us, 300 x 100 x 1500 1345 -> 752
// us, 1024 x 64 x 2000 7.05 -> 6.00 ms (int8 samples 5.64 -> 4.79).  Loading a
// row's chunks by neighbouring lanes (padded LDS rows) was 1 % faster on float
// samples and 2 % slower on int8 ones.
//
// LDS rows: a block's R rows lie in R / 2 chunks of two samples (16 bytes), chunk
// q of every block side by side, so that the 16 blocks a wave reads at once are
// one run of 256 bytes (a block's rows side by side would put them 32 bytes
// apart, on half of the banks).  Each thread writes the LDS position of its
// own number and loads whichever row belongs there.
// Integer-valued samples give exact sums while they stay below 2^24 (checked
// on the host).  Im of autos is written as exactly zero.
#include "common.h"
#include "launch.h"

namespace corr {

constexpr int kF32BT = 64;  // inputs per panel
constexpr int kF32KS = 16;  // samples per LDS stage

template <typename T>
struct SampleTraits;
template <>
struct SampleTraits<float2> {
  static constexpr int kBytes = 8;
  static constexpr int kPerChunk = 2;   // samples per 16-byte global load
};
template <>
struct SampleTraits<int8_t> {
  static constexpr int kBytes = 2;
  static constexpr int kPerChunk = 8;
};

// 16-byte chunk of samples t .. t+P-1 of one row of which those before t1 lie
// in the pass, zero elsewhere (the last stage of a pass).
template <typename S>
__device__ __forceinline__ int4 load_part(const int8_t* __restrict__ row, int64_t t, int64_t t1) {
  constexpr int P = SampleTraits<S>::kPerChunk;
  constexpr int B = SampleTraits<S>::kBytes;
  const int8_t* p = row + t * B;
  if (t + P <= t1) return load16_any<int4>(p);
  int w[4] = {0, 0, 0, 0};
#pragma unroll
  for (int s = 0; s < P; ++s) {
    if (t + s < t1) {
      if constexpr (B == 8) {
        const int* f = reinterpret_cast<const int*>(p + 8 * s);
        w[2 * s] = f[0];
        w[2 * s + 1] = f[1];
      } else {
        const uint32_t h = *reinterpret_cast<const uint16_t*>(p + 2 * s);
        w[s >> 1] |= (int)(h << (16 * (s & 1)));
      }
    }
  }
  return make_int4(w[0], w[1], w[2], w[3]);
}

// Raw chunk -> P float2 samples (exact for int8).
template <typename S>
__device__ __forceinline__ void unpack(int4 raw, float2 (&v)[SampleTraits<S>::kPerChunk]) {
  constexpr int B = SampleTraits<S>::kBytes;
  const int ws[4] = {raw.x, raw.y, raw.z, raw.w};
  if constexpr (B == 8) {
    v[0] = make_float2(__int_as_float(ws[0]), __int_as_float(ws[1]));
    v[1] = make_float2(__int_as_float(ws[2]), __int_as_float(ws[3]));
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[2 * q] = make_float2((float)(int8_t)(ws[q] & 0xFF), (float)(int8_t)((ws[q] >> 8) & 0xFF));
      v[2 * q + 1] = make_float2((float)(int8_t)((ws[q] >> 16) & 0xFF), (float)(int8_t)((ws[q] >> 24) & 0xFF));
    }
  }
}

// acc += a conj(b): re = ar br + ai bi, im = ai br - ar bi.
__device__ __forceinline__ void f32_cmac(float& vr, float& vi, float2 a, float2 b) {
  vr = fmaf(a.x, b.x, vr);
  vr = fmaf(a.y, b.y, vr);
  vi = fmaf(a.y, b.x, vi);
  vi = fmaf(-a.x, b.y, vi);
}

__device__ __forceinline__ void f32_put(const XArgs& a, float2* __restrict__ out, int i, int j, float re, float im) {
  if (i < a.n_in && j <= i) {
    float2* p = out + tri_index(i, j);
    if (i == j) im = 0.f;
    if (a.accumulate) {
      float2 o = *p;
      o.x += re;
      o.y += im;
      *p = o;
    } else {
      *p = make_float2(re, im);
    }
  }
}

// Two neighbouring products (i, j), (i, j + 1): one 16-byte store where both
// exist and are only stored.
__device__ __forceinline__ void f32_put2(const XArgs& a, float2* __restrict__ out, int i, int j, float re0, float im0,
                                         float re1, float im1) {
  if (!a.accumulate && i < a.n_in && j + 1 < i) {
    const float4 v = make_float4(re0, im0, re1, im1);
    __builtin_memcpy(out + tri_index(i, j), &v, 16);
  } else {
    f32_put(a, out, i, j, re0, im0);
    f32_put(a, out, i, j + 1, re1, im1);
  }
}

// DIAG: the diagonal tiles (ch0, I0) and (ch1, I1) (two_ok: the second exists,
// else it repeats the first and is not stored); else the tile (I0, I1) of
// channel ch0 = ch1.  Stages that lie wholly inside the pass are loaded 16
// bytes at a time, unconditionally (so the compiler does not wait for them
// before the FMAs that follow); only the last, partial stage checks its
// samples.  Rows past N_I are read from a clamped row and only reach products
// that are never stored.
// SUB 32 or 16: the panels are those of 128 / SUB channels from ch0 of at most SUB
// inputs, SUB rows each; every wave takes 32 / SUB of them, a lane one block.
template <typename S, bool DIAG, int SUB>
__device__ __forceinline__ void xeng_f32_tile(const XArgs& a, float2 (*lds)[2][kF32KS][kF32BT], int split, int ch0, int I0,
                                              int ch1, int I1, bool two_ok) {
  constexpr int BT = kF32BT;
  constexpr int P = SampleTraits<S>::kPerChunk;
  constexpr int B = SampleTraits<S>::kBytes;
  constexpr int CPR = kF32KS / P;            // chunks per row per stage
  constexpr int CHUNKS = BT * CPR;           // per panel
  constexpr int LPT = (CHUNKS + 255) / 256;  // chunks per thread per panel
  constexpr int R = BT / 16;                 // rows (and cols) per thread
  constexpr bool TWO = DIAG && SUB == BT;    // a pair of diagonal tiles
  constexpr int NX = R * R / 16;             // products of the second tile's diagonal blocks per thread (TWO)
  constexpr int PER = BT / SUB;              // channels per panel (DIAG)

  const int64_t n_t = a.k_bytes / B;
  const int64_t split_t = a.k_split_bytes / B;
  const int64_t t0 = (int64_t)split * split_t;
  const int64_t t1 = min(n_t, t0 + split_t);
  const int n_st = t1 > t0 ? (int)((t1 - t0 + kF32KS - 1) / kF32KS) : 0;
  const int n_full = t1 > t0 ? (int)((t1 - t0) / kF32KS) : 0;

  const int tid = threadIdx.x;
  const int tx = tid & 15, ty = tid >> 4;

  // This thread's LDS position and the panel row that belongs there.
  const int pos = tid % BT;
  const int prow = (pos % 32) / 2 * R + pos / 32 * 2 + pos % 2;
  const int kc0 = tid / BT;                  // its first chunk; the next ones follow 256 / BT apart
  const int8_t* __restrict__ x = static_cast<const int8_t*>(a.x);
  const int cha = SUB == BT ? ch0 : min(ch0 + prow / SUB, a.n_ch - 1);
  const int chb = SUB == BT ? ch1 : min(ch0 + PER + prow / SUB, a.n_ch - 1);
  const int8_t* pa = x + (int64_t)cha * a.ch_stride_b + (int64_t)min(I0 * BT + prow % SUB, a.n_in - 1) * a.row_stride_b;
  const int8_t* pb = x + (int64_t)chb * a.ch_stride_b + (int64_t)min(I1 * BT + prow % SUB, a.n_in - 1) * a.row_stride_b;

  int4 ga[LPT], gb[LPT];
  auto gload = [&](int st) {
    if (CHUNKS < 256 && tid >= CHUNKS) return;
    const int64_t ts = t0 + (int64_t)st * kF32KS;
    if (st < n_full) {
#pragma unroll
      for (int q = 0; q < LPT; ++q) {
        const int64_t o = (ts + (kc0 + 256 / BT * q) * P) * B;
        ga[q] = load16_any<int4>(pa + o);
        gb[q] = load16_any<int4>(pb + o);
      }
    } else {
#pragma unroll
      for (int q = 0; q < LPT; ++q) {
        const int64_t t = ts + (kc0 + 256 / BT * q) * P;
        ga[q] = load_part<S>(pa, t, t1);
        gb[q] = load_part<S>(pb, t, t1);
      }
    }
  };
  auto lstore = [&](int buf) {
    if (CHUNKS < 256 && tid >= CHUNKS) return;
#pragma unroll
    for (int q = 0; q < LPT; ++q) {
      const int k = (kc0 + 256 / BT * q) * P;
      float2 v[P];
      unpack<S>(ga[q], v);
#pragma unroll
      for (int s = 0; s < P; ++s) lds[buf][0][k + s][pos] = v[s];
      unpack<S>(gb[q], v);
#pragma unroll
      for (int s = 0; s < P; ++s) lds[buf][1][k + s][pos] = v[s];
    }
  };

  // This thread's block: rows rb against columns cb, DIAG: of tile u.
  int rb = ty, cb = tx;
  const int u = DIAG ? tid >> 7 : 0;
  // SUB: of channel sub of the panel, none past the last of the wave's channels.
  constexpr int NSB = SUB / R, NBL = NSB * (NSB + 1) / 2;   // blocks per side and in all
  const int sc = (tid & 63) / NBL;
  const int sub = (tid >> 6 & 1) * (32 / SUB) + min(sc, 32 / SUB - 1);
  if (DIAG && SUB < BT) {
    const int t = (tid & 63) % NBL;
    if (t < NBL - NSB) {
      tile_decode(t, rb, cb);
      ++rb;
    } else {
      rb = cb = t - (NBL - NSB);
    }
    rb += sub * NSB;
    cb += sub * NSB;
  } else if (DIAG) {
    const int t = tid & 127;
    if (t < 120) {
      tile_decode(t, rb, cb);
      ++rb;
    } else {
      rb = cb = t - 120;
    }
  }
  // DIAG: row xr against columns xc .. xc + NX - 1 of diagonal block xb of tile u.
  const int xb = 8 + (ty & 7);
  const int xr = tx * NX / R, xc = tx * NX % R;
  const int xpr = xr / 2 * 32 + 2 * xb + xr % 2;

  float vr[R][R], vi[R][R], er[TWO ? NX : 1], ei[TWO ? NX : 1];
#pragma unroll
  for (int m = 0; m < R; ++m)
#pragma unroll
    for (int n = 0; n < R; ++n) vr[m][n] = vi[m][n] = 0.f;
#pragma unroll
  for (int n = 0; n < (TWO ? NX : 1); ++n) er[n] = ei[n] = 0.f;

  if (n_st > 0) {
    gload(0);
    lstore(0);
  }
  __syncthreads();
  for (int st = 0; st < n_st; ++st) {
    const int cur = st & 1;
    if (st + 1 < n_st) gload(st + 1);
    const float2 (*As)[BT] = lds[cur][u];
    const float2 (*Bs)[BT] = DIAG ? As : lds[cur][1];
#pragma unroll 4
    for (int k = 0; k < kF32KS; ++k) {
      float2 av[R], bv[R];
#pragma unroll
      for (int q = 0; q < R / 2; ++q)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          av[2 * q + e] = As[k][32 * q + 2 * rb + e];
          bv[2 * q + e] = Bs[k][32 * q + 2 * cb + e];
        }
#pragma unroll
      for (int m = 0; m < R; ++m)
#pragma unroll
        for (int n = 0; n < R; ++n) f32_cmac(vr[m][n], vi[m][n], av[m], bv[n]);
      if constexpr (TWO) {
        const float2 xa = As[k][xpr];
#pragma unroll
        for (int n = 0; n < NX; ++n)
          f32_cmac(er[n], ei[n], xa, As[k][(xc + n) / 2 * 32 + 2 * xb + (xc + n) % 2]);
      }
    }
    if (st + 1 < n_st) lstore(cur ^ 1);
    __syncthreads();
  }

  float2* const base = static_cast<float2*>(a.out) + (int64_t)split * a.out_split_stride;
  if (u == 1 && !two_ok) return;
  const int ch = SUB < BT ? ch0 + u * PER + sub : u ? ch1 : ch0;
  if (SUB < BT && (sc >= 32 / SUB || ch >= a.n_ch)) return;
  float2* out = base + (int64_t)ch * a.n_products;
  // first row, first column of the tile
  const int ti = SUB < BT ? -sub * SUB : (u ? I1 : I0) * BT, tj = DIAG ? ti : I1 * BT;
#pragma unroll
  for (int m = 0; m < R; ++m)
#pragma unroll
    for (int n = 0; n < R; n += 2)
      f32_put2(a, out, ti + rb * R + m, tj + cb * R + n, vr[m][n], vi[m][n], vr[m][n + 1], vi[m][n + 1]);
  if constexpr (TWO) {
#pragma unroll
    for (int n = 0; n < NX; ++n)
      f32_put(a, out, ti + xb * R + xr, ti + xb * R + xc + n, er[n], ei[n]);
  }
}

// Items of a split: the pairs of diagonal tiles (channel-major), then the
// off-diagonal tiles of each channel.
template <typename S, int SUB>
__global__ __launch_bounds__(256, 4) void xeng_f32_kernel(XArgs a) {
  __shared__ __attribute__((aligned(16))) float2 lds[2][2][kF32KS][kF32BT];
  const int64_t slot = blockIdx.x / kNumXcd;
  const int64_t item = xcd_item(blockIdx.x, a.per_xcd);
  if (slot >= a.per_xcd || item >= a.n_items) return;
  const int nb = (a.n_in + kF32BT - 1) / kF32BT;
  const int n_diag = a.n_ch * nb;            // diagonal tiles
  const int per_split = a.n_items / a.n_split;
  const int split = (int)(item / per_split);
  const int v = (int)(item % per_split);
  if constexpr (SUB < kF32BT) {
    xeng_f32_tile<S, true, SUB>(a, lds, split, v * (128 / SUB), 0, 0, 0, true);
  } else if (v < (n_diag + 1) / 2) {
    const int d0 = 2 * v, d1 = min(2 * v + 1, n_diag - 1);
    xeng_f32_tile<S, true, kF32BT>(a, lds, split, d0 / nb, d0 % nb, d1 / nb, d1 % nb, d1 != d0);
  } else {
    const int o = v - (n_diag + 1) / 2;
    const int n_off = nb * (nb - 1) / 2;
    int I, J;
    tile_decode(o % n_off, I, J);            // (I + 1, J): strictly lower
    xeng_f32_tile<S, false, kF32BT>(a, lds, split, o / n_off, I + 1, o / n_off, J, true);
  }
}

// sample_bytes: 8 (complex float32) or 2 (complex int8); sub: rows a channel has in
// a panel (64, or 32 or 16 where a channel has no more inputs).
hipError_t launch_xeng_f32(const XArgs& a, int sample_bytes, int sub, hipStream_t s) {
  const int64_t grid = (int64_t)a.per_xcd * kNumXcd;
  if (grid <= 0) return hipSuccess;
#define CORR_F32(S, SUB) hipLaunchKernelGGL((xeng_f32_kernel<S, SUB>), dim3((unsigned)grid), dim3(256), 0, s, a)
  if (sample_bytes == 8) {
    if (sub == 64) CORR_F32(float2, 64); else if (sub == 32) CORR_F32(float2, 32); else CORR_F32(float2, 16);
  } else {
    if (sub == 64) CORR_F32(int8_t, 64); else if (sub == 32) CORR_F32(int8_t, 32); else CORR_F32(int8_t, 16);
  }
#undef CORR_F32
  return hipGetLastError();
}

}  // namespace corr
