// int8 matrix-core X-engine for sample rows that are not 16-byte aligned (a
// contiguous array with an odd number of samples, a row stride that is not a
// multiple of 8, an offset into a longer record): V_ij[c] += sum_t x_i[c,t]
// conj(x_j[c,t]) for complex int8 samples, int32 accumulation (exact within
// the host-checked bound).
//
// The products are those of the aligned engine (xengine_mfma.hip): with each
// row as interleaved (re, im) bytes along K = 2T, Re V = A B^T and Im V =
// (-iA) B^T with -iA = (im, -re) made in registers, as 16 x 16 x 64 MFMAs
// over the lower-triangle tiles of Fig. 2's outer product.  Only the staging
// differs.  The aligned engine's loads go straight into LDS and need 16-byte
// aligned addresses; here every lane loads its 16 bytes from wherever the row
// starts (any even address) into registers, PF stages ahead, and writes them
// to LDS in the aligned engine's layout, so the shift costs no instruction.
// Two LDS stage buffers and one barrier per stage: the barrier of stage s + 1
// follows every wave's completed reads of stage s, whose buffer then takes
// stage s + 2.
//
// Bound: as the aligned engine (matrix cores and the L2-to-LDS traffic).  The
// extra register stop costs 18 % against it: 1024 inputs x 96 channels x 8001
// samples take 2.00 ms, 8000 samples (aligned rows) 1.69 ms, and 12.5 ms when
// the samples were loaded two bytes at a time; 231 x 524 x 2866 takes 373 us
// (1948 before; 403 with a condition around the loads of the steady loop), 100
// x 133 x 2001 58 us with its read-out (125 before).  Two
// stages in flight fill the registers of two waves per SIMD (254 VGPRs);
// writing the LDS stage after the fragment reads instead of before was 1 %
// slower.
#include <type_traits>

#include "common.h"
#include "launch.h"

namespace corr {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kUKC = 64;   // K bytes (32 samples) per stage

// 16-byte chunk c (0..3) of LDS row r lives at chunk c ^ uswz(r).
__device__ __forceinline__ int uswz(int r) { return (r >> 2) & 3; }

// Multiply two packed complex int8 samples by -i: (re, im) -> (im, -re).
// |re| <= 127, so the negation never overflows.
__device__ __forceinline__ int umul_mi(int w) {
  const uint32_t u = (uint32_t)w;
  const uint32_t neg = 0x01000100u - (u & 0x00FF00FFu);   // low byte of each 16-bit lane = -re
  return (int)__builtin_amdgcn_perm(neg, u, 0x06030401u);
}

// The up to 16 bytes of a row at p of which the first `valid` (even) lie in
// the pass, zero elsewhere.
__device__ __forceinline__ v4i load_part(const int8_t* p, int64_t valid) {
  v4i v = {0, 0, 0, 0};
  if (valid >= 16) {
    v = load16_any<v4i>(p);
  } else {
    const uint16_t* h = reinterpret_cast<const uint16_t*>(p);
#pragma unroll
    for (int s = 0; s < 8; ++s)
      if (2 * s < valid) v[s >> 1] |= (int)((uint32_t)h[s] << (16 * (s & 1)));
  }
  return v;
}

// One BT x BT tile (I, J) of one channel over one K split.  Four waves
// (2 x 2), each (BT / 2) x (BT / 2) as NB x NB blocks of 16 x 16.  DIAG tiles
// stage one panel that serves as both operands; there the wave of the strictly
// upper quarter only loads, and the diagonal waves skip their strictly upper
// blocks.
template <int BT, bool DIAG>
__device__ __forceinline__ void xeng_i8u_tile(const XArgs& a, int8_t* lds, int ch, int split, int I, int J) {
  constexpr int WT = BT / 2;
  constexpr int NB = WT / 16;
  constexpr int QPW = BT / 64;               // 1 KB (16-row) pieces per operand and wave
  constexpr int NOP = DIAG ? 1 : 2;
  constexpr int PANEL = BT * kUKC;
  constexpr int STAGE = PANEL * NOP;
  constexpr int PF = BT == 128 ? 2 : 4;      // stages in flight in registers
  static_assert(PF == 2 || PF == 4, "the unrolled loop below");

  const int8_t* __restrict__ xc = static_cast<const int8_t*>(a.x) + (int64_t)ch * a.ch_stride_b;
  const int64_t k0 = (int64_t)split * a.k_split_bytes;
  const int64_t k1 = min(a.k_bytes, k0 + a.k_split_bytes);
  const int n_st = k1 > k0 ? (int)((k1 - k0 + kUKC - 1) / kUKC) : 0;
  // Stages whose 64 bytes all lie in [k0, k1) and whose offsets fit 32 bits.
  const int n_fast = a.row_stride_b < (int64_t(1) << 24) ? (int)((k1 - k0) / kUKC) : 0;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  // This lane's part of each piece: LDS row lane / 4 (of 16), LDS chunk lane
  // % 4, which holds the row's chunk (lane % 4) ^ uswz.
  const int8_t* const tA = xc + (int64_t)(I * BT) * a.row_stride_b + k0;
  const int8_t* const tB = xc + (int64_t)(J * BT) * a.row_stride_b + k0;
  uint32_t off[NOP][QPW];
#pragma unroll
  for (int q = 0; q < QPW; ++q) {
    const int r = (wave * QPW + q) * 16 + (lane >> 2);
    const int c = (lane & 3) ^ uswz(r);
    off[0][q] = (uint32_t)((int64_t)(min(I * BT + r, a.n_in - 1) - I * BT) * a.row_stride_b + 16 * c);
    if constexpr (!DIAG) off[1][q] = (uint32_t)((int64_t)(min(J * BT + r, a.n_in - 1) - J * BT) * a.row_stride_b + 16 * c);
  }

  v4i R[PF][NOP][QPW];
  auto gload_full = [&](auto S, int st) {   // st < n_fast
    constexpr int sl = decltype(S)::value;
#pragma unroll
    for (int q = 0; q < QPW; ++q)
#pragma unroll
      for (int o = 0; o < NOP; ++o)
        R[sl][o][q] = load16_any<v4i>((o == 0 ? tA : tB) + (int64_t)st * kUKC + off[o][q]);
  };
  auto gload = [&](auto S, int st) {
    constexpr int sl = decltype(S)::value;
    if (st < n_fast) {
      gload_full(S, st);
    } else {
#pragma unroll
      for (int q = 0; q < QPW; ++q) {
        const int r = (wave * QPW + q) * 16 + (lane >> 2);
        const int64_t kk = k0 + (int64_t)st * kUKC + 16 * ((lane & 3) ^ uswz(r));
#pragma unroll
        for (int o = 0; o < NOP; ++o) {
          const int64_t row = min((o == 0 ? I : J) * BT + r, a.n_in - 1);
          R[sl][o][q] = load_part(xc + row * a.row_stride_b + kk, k1 - kk);
        }
      }
    }
  };
  auto lstore = [&](auto S, int st) {
    constexpr int sl = decltype(S)::value;
    int8_t* base = lds + (st & 1) * STAGE + wave * QPW * 1024 + lane * 16;
#pragma unroll
    for (int q = 0; q < QPW; ++q)
#pragma unroll
      for (int o = 0; o < NOP; ++o) *reinterpret_cast<v4i*>(base + o * PANEL + q * 1024) = R[sl][o][q];
  };
  // This wave's LDS accesses are done, then every wave's (loads stay in flight).
  auto barrier = [&] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

  v4i vr[NB][NB], vi[NB][NB];
#pragma unroll
  for (int m = 0; m < NB; ++m)
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      vr[m][n] = v4i{0, 0, 0, 0};
      vi[m][n] = v4i{0, 0, 0, 0};
    }

  auto read = [&](int st, v4i (&af)[NB], v4i (&bf)[NB]) {
    const int8_t* As = lds + (st & 1) * STAGE;
    const int8_t* Bs = DIAG ? As : As + PANEL;
    const int c = lane >> 4;
#pragma unroll
    for (int m = 0; m < NB; ++m) {
      const int r = wm * WT + m * 16 + (lane & 15);
      af[m] = *reinterpret_cast<const v4i*>(As + r * kUKC + 16 * (c ^ uswz(r)));
    }
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const int r = wn * WT + n * 16 + (lane & 15);
      bf[n] = *reinterpret_cast<const v4i*>(Bs + r * kUKC + 16 * (c ^ uswz(r)));
    }
  };
  auto compute = [&](auto sk, const v4i (&af)[NB], const v4i (&bf)[NB]) {
    constexpr bool SK = decltype(sk)::value;
#pragma unroll
    for (int m = 0; m < NB; ++m)
#pragma unroll
      for (int n = 0; n < NB; ++n)
        if (!(SK && n > m)) vr[m][n] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[m], bf[n], vr[m][n], 0, 0, 0);
#pragma unroll
    for (int m = 0; m < NB; ++m) {
      v4i ra;
#pragma unroll
      for (int q = 0; q < 4; ++q) ra[q] = umul_mi(af[m][q]);
#pragma unroll
      for (int n = 0; n < NB; ++n)
        if (!(SK && n > m)) vi[m][n] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ra, bf[n], vi[m][n], 0, 0, 0);
    }
  };

  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  using S2 = std::integral_constant<int, PF == 4 ? 2 : 0>;
  using S3 = std::integral_constant<int, PF == 4 ? 3 : 1>;
  // Stage st waits in register slot st % PF.  Iteration s moves stage s + 2 to
  // LDS, refills its slot with stage s + 2 + PF, reads the fragments of stage
  // s + 1 and multiplies those of stage s.  FULL: all of these exist and the
  // loaded ones lie wholly in the pass.  Without any condition around a load the
  // compiler waits for the oldest stage only (vmcnt counts what was issued
  // since); with one it waits for all of them.
  // (64-row tiles gain nothing from it and would spill.)
  const bool deep = BT == 128 && n_fast > 2 * PF + 1;
  if (deep) {
    gload_full(S0{}, 0);
    gload_full(S1{}, 1);
    if constexpr (PF == 4) {
      gload_full(S2{}, 2);
      gload_full(S3{}, 3);
    }
    lstore(S0{}, 0);
    gload_full(S0{}, PF);
    barrier();
    lstore(S1{}, 1);
    gload_full(S1{}, 1 + PF);
  } else {
    if (0 < n_st) gload(S0{}, 0);
    if (1 < n_st) gload(S1{}, 1);
    if constexpr (PF == 4) {
      if (2 < n_st) gload(S2{}, 2);
      if (3 < n_st) gload(S3{}, 3);
    }
    if (0 < n_st) lstore(S0{}, 0);
    if (PF < n_st) gload(S0{}, PF);
    barrier();
    if (1 < n_st) lstore(S1{}, 1);
    if (1 + PF < n_st) gload(S1{}, 1 + PF);
  }
  auto run = [&](auto sk, auto active) {
    constexpr bool ACT = decltype(active)::value;
    v4i af0[NB], bf0[NB], af1[NB], bf1[NB];
    if (ACT && n_st > 0) read(0, af0, bf0);
    auto step = [&](auto full, auto U, int s) {
      constexpr bool FULL = decltype(full)::value;
      if (FULL || s + 1 < n_st) {
        barrier();
        if (FULL || s + 2 < n_st) {
          lstore(U, s + 2);
          if constexpr (FULL) gload_full(U, s + 2 + PF);
          else if (s + 2 + PF < n_st) gload(U, s + 2 + PF);
        }
        if constexpr (ACT) read(s + 1, af1, bf1);
      }
      if constexpr (ACT) {
        compute(sk, af0, bf0);
#pragma unroll
        for (int m = 0; m < NB; ++m) {
          af0[m] = af1[m];
          bf0[m] = bf1[m];
        }
      }
    };
    auto steps = [&](auto full, int s) {   // stage s + 2 + u waits in slot (2 + u) % PF
      constexpr bool FULL = decltype(full)::value;
      step(full, std::integral_constant<int, 2 % PF>{}, s);
      if (FULL || s + 1 < n_st) step(full, std::integral_constant<int, 3 % PF>{}, s + 1);
      if constexpr (PF == 4) {
        if (FULL || s + 2 < n_st) step(full, S0{}, s + 2);
        if (FULL || s + 3 < n_st) step(full, S1{}, s + 3);
      }
    };
    int s = 0;
    if (deep)
      for (; s + 2 * PF + 1 < n_fast; s += PF) steps(std::true_type{}, s);
    for (; s < n_st; s += PF) steps(std::false_type{}, s);
  };
  if (DIAG && wm < wn) {
    run(std::false_type{}, std::false_type{});
    return;
  }
  if (DIAG && wm == wn) run(std::true_type{}, std::true_type{});
  else run(std::false_type{}, std::true_type{});

  // Epilogue.  16 x 16 accumulator layout: register r of lane l holds row
  // 4*(l/16) + r, column l%16.
  int2* __restrict__ out = static_cast<int2*>(a.out) + (int64_t)split * a.out_split_stride +
                           (int64_t)ch * a.n_products;
#pragma unroll
  for (int m = 0; m < NB; ++m)
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const int j = J * BT + wn * WT + n * 16 + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = I * BT + wm * WT + m * 16 + 4 * (lane >> 4) + r;
        if (i < a.n_in && j <= i) {
          int2* p = out + tri_index(i, j);
          const int re = vr[m][n][r];
          const int im = (i == j) ? 0 : vi[m][n][r];
          if (a.accumulate) {
            int2 o = *p;
            o.x += re;
            o.y += im;
            *p = o;
          } else {
            *p = make_int2(re, im);
          }
        }
      }
    }
}

template <int BT>
__global__ __launch_bounds__(256, BT == 128 ? 2 : 4) void xeng_i8u_kernel(XArgs a) {
  __shared__ __attribute__((aligned(1024))) int8_t lds[2 * 2 * BT * kUKC];
  const int64_t slot = blockIdx.x / kNumXcd;
  const int64_t item = xcd_item(blockIdx.x, a.per_xcd);
  if (slot >= a.per_xcd || item >= a.n_items) return;
  int ch, split, I, J;
  item_decode(a, item, ch, split, I, J);
  if (I == J) xeng_i8u_tile<BT, true>(a, lds, ch, split, I, J);
  else xeng_i8u_tile<BT, false>(a, lds, ch, split, I, J);
}

hipError_t launch_xeng_i8u(const XArgs& a, int bt, hipStream_t s) {
  const int64_t grid = (int64_t)a.per_xcd * kNumXcd;
  if (grid <= 0) return hipSuccess;
  if (bt == 128) hipLaunchKernelGGL((xeng_i8u_kernel<128>), dim3((unsigned)grid), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((xeng_i8u_kernel<64>), dim3((unsigned)grid), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace corr
