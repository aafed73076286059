// Accumulator maintenance: ordered reduction of K-split partial tiles into the
// integration accumulator, the FP64 long-run fold, and fills.
//
// Fig. 1: the accumulators are read after an interval, divided by the number
// of updates (left to the caller, who gets the raw sums and the count) and
// reset.  The long-run fold keeps L += V in FP64 across many integrations.
#include "common.h"
#include "launch.h"

namespace corr {

// acc[k] = (accumulate ? acc[k] : 0) + part[0][k] + part[1][k] + ... in that
// order (integer sums are exact; the fixed order keeps float sums
// reproducible).  n = number of (re, im) pairs per partial buffer.  A thread
// takes two neighbouring pairs (wide: one 16-byte load per split, when n is
// even and both buffers are 16-byte aligned) and issues the loads of four
// splits before adding them in split order, so several loads are in flight
// per thread.
template <typename T2>
struct Wide;
template <>
struct Wide<int2> { typedef int4 T; };
template <>
struct Wide<float2> { typedef float4 T; };

template <typename T4>
__device__ __forceinline__ void add4(T4& s, const T4& p) {
  s.x += p.x;
  s.y += p.y;
  s.z += p.z;
  s.w += p.w;
}

template <typename T2>
__global__ void reduce_splits_kernel(const T2* __restrict__ part, int64_t n, int n_split,
                                     T2* __restrict__ acc, int accumulate, int wide) {
  using T4 = typename Wide<T2>::T;
  const int64_t k = 2 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);   // first pair
  if (k >= n) return;
  if (wide) {
    const T4* __restrict__ p4 = reinterpret_cast<const T4*>(part);
    const int64_t n4 = n / 2, k4 = k / 2;
    T4 s = p4[k4];
    int q = 1;
    for (; q + 3 < n_split; q += 4) {
      const T4 a = p4[(int64_t)q * n4 + k4], b = p4[(int64_t)(q + 1) * n4 + k4];
      const T4 c = p4[(int64_t)(q + 2) * n4 + k4], d = p4[(int64_t)(q + 3) * n4 + k4];
      add4(s, a);
      add4(s, b);
      add4(s, c);
      add4(s, d);
    }
    for (; q < n_split; ++q) add4(s, p4[(int64_t)q * n4 + k4]);
    T4* __restrict__ a4 = reinterpret_cast<T4*>(acc);
    if (accumulate) {
      T4 o = a4[k4];
      add4(o, s);   // o + s: the same operand order as the pair path below
      s = o;
    }
    a4[k4] = s;
    return;
  }
  for (int64_t kk = k; kk < min(k + 2, n); ++kk) {   // pair by pair
    T2 s = part[kk];
    for (int q = 1; q < n_split; ++q) {
      const T2 p = part[(int64_t)q * n + kk];
      s.x += p.x;
      s.y += p.y;
    }
    if (accumulate) {
      const T2 o = acc[kk];
      s.x = o.x + s.x;
      s.y = o.y + s.y;
    }
    acc[kk] = s;
  }
}

__global__ void fill_zero_kernel(uint4* __restrict__ p, int64_t n16) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n16) p[k] = make_uint4(0u, 0u, 0u, 0u);
}

static inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

hipError_t launch_reduce_splits(const void* part, int64_t n_pairs, int n_split, void* acc, int accumulate,
                                bool is_int, hipStream_t s) {
  if (n_pairs <= 0) return hipSuccess;
  // two pairs per thread
  const int64_t threads = (n_pairs + 1) / 2;
  const int wide = (n_pairs % 2 == 0) && (((reinterpret_cast<uintptr_t>(part) | reinterpret_cast<uintptr_t>(acc)) & 15) == 0);
  if (is_int)
    hipLaunchKernelGGL(reduce_splits_kernel<int2>, dim3(grid_for(threads, 256)), dim3(256), 0, s,
                       static_cast<const int2*>(part), n_pairs, n_split, static_cast<int2*>(acc), accumulate, wide);
  else
    hipLaunchKernelGGL(reduce_splits_kernel<float2>, dim3(grid_for(threads, 256)), dim3(256), 0, s,
                       static_cast<const float2*>(part), n_pairs, n_split, static_cast<float2*>(acc), accumulate,
                       wide);
  return hipGetLastError();
}

// Zero `bytes` (a multiple of 16) at a 16-byte aligned device pointer.
hipError_t launch_fill_zero(void* p, int64_t bytes, hipStream_t s) {
  const int64_t n16 = bytes / 16;
  if (n16 <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(grid_for(n16, 256)), dim3(256), 0, s, static_cast<uint4*>(p), n16);
  return hipGetLastError();
}

// Any address and length (a kernel, not a memset node, also under stream capture).
__global__ void fill_zero_bytes_kernel(uint8_t* __restrict__ p, int64_t n) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) p[k] = 0;
}

hipError_t launch_fill_zero_bytes(void* p, int64_t bytes, hipStream_t s) {
  if (bytes <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_zero_bytes_kernel, dim3(grid_for(bytes, 256)), dim3(256), 0, s, static_cast<uint8_t*>(p),
                     bytes);
  return hipGetLastError();
}

// Guard word w of band g: a position-dependent pattern, so that a band copied
// or shifted onto another is also seen.
__device__ __forceinline__ uint32_t guard_word(int g, int w) {
  return 0xA5C3F00Du ^ ((uint32_t)(g * (kGuardBytes / 4) + w) * 0x9E3779B1u);
}

__global__ void guard_fill_kernel(uint8_t* __restrict__ ws, GuardList gl) {
  const int g = blockIdx.x, w = threadIdx.x;   // one block per band, one thread per word
  reinterpret_cast<uint32_t*>(ws + gl.off[g])[w] = guard_word(g, w);
}

// One workgroup: compare the bands with the pattern; *bad is 0 if no word
// differs, else the number of threads that saw one that does.
__device__ __forceinline__ void guard_check(const uint8_t* __restrict__ ws, const GuardList& gl,
                                            uint32_t* __restrict__ bad) {
  constexpr int kWords = kGuardBytes / 4;
  uint32_t n = 0;
  for (int k = threadIdx.x; k < gl.n * kWords; k += blockDim.x) {
    const int g = k / kWords, w = k % kWords;
    n += reinterpret_cast<const uint32_t*>(ws + gl.off[g])[w] != guard_word(g, w) ? 1u : 0u;
  }
  const int found = __syncthreads_count(n != 0);   // threads that saw a difference
  if (threadIdx.x == 0) *bad = (uint32_t)found;
}

// A dump in one launch, with the check's result written to mapped host memory
// (as separate copies, fold, check and read-back of the check's word it was up
// to five queue entries of 2 to 6 us each: the call took 27 us for 4.6 KB on
// the device, 39 us to the host, now 15 and 16).
// Workgroup 0 checks the bands when ws is given; the others take 4 scalars a
// thread: one 16-byte piece of the integration, or two pairs of scalars where
// the long-run sum takes part, and one pair where it only takes the integration
// in (512 inputs x 256 channels: 251 us with 4 scalars a thread, 239 with 2).
// Bound: HBM, each buffer touched once: a 3.2 GB integration is read out 0.28 ms
// sooner than by the runtime's device copy (1.28 ms, 5 TB/s read + written).
// dst may have any 4-byte alignment.
template <typename T, int MODE>
__global__ __launch_bounds__(256) void dump_kernel(const T* __restrict__ acc, double* __restrict__ L,
                                                   void* __restrict__ dst, int64_t n, const uint8_t* __restrict__ ws,
                                                   GuardList gl, uint32_t* __restrict__ bad) {
  constexpr bool kV = MODE != kDumpCopyLong && MODE != kDumpCheck;                // reads acc
  constexpr bool kL = MODE == kDumpCopyLong || MODE >= kDumpFold;                 // reads L
  constexpr bool kFold = MODE >= kDumpFold;
  typedef T T4 __attribute__((ext_vector_type(4)));
  typedef double D2 __attribute__((ext_vector_type(2)));
  int64_t b = blockIdx.x;
  if (ws != nullptr) {
    if (b == 0) {
      guard_check(ws, gl, bad);
      return;
    }
    --b;
  }
  if constexpr (kL) {
    // pairs, so that neighbouring lanes touch neighbouring 16 bytes of the sum
    typedef T T2 __attribute__((ext_vector_type(2)));
    constexpr int G = MODE == kDumpFold ? 1 : 2;
    const int64_t k = b * (512 * G) + 2 * threadIdx.x;
    T2 v[G] = {};
    D2 l[G] = {};
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (k + 512 * g < n) {               // n is even
        if constexpr (kV) v[g] = *reinterpret_cast<const T2*>(acc + k + 512 * g);
        l[g] = *reinterpret_cast<const D2*>(L + k + 512 * g);
      }
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (k + 512 * g < n) {
        const int64_t q = k + 512 * g;
        if constexpr (kFold) {
          l[g] += D2{(double)v[g][0], (double)v[g][1]};
          *reinterpret_cast<D2*>(L + q) = l[g];
        }
        if constexpr (MODE == kDumpFoldCopy) __builtin_memcpy(static_cast<T*>(dst) + q, &v[g], 8);
        else if constexpr (MODE != kDumpFold) __builtin_memcpy(static_cast<double*>(dst) + q, &l[g], 16);
      }
  } else if constexpr (MODE == kDumpCopy) {
    const int64_t k = 4 * (b * 256 + threadIdx.x);
    if (k + 4 <= n) {
      const T4 v = *reinterpret_cast<const T4*>(acc + k);
      __builtin_memcpy(static_cast<T*>(dst) + k, &v, 16);
    } else {
      for (int64_t q = k; q < n; ++q) __builtin_memcpy(static_cast<T*>(dst) + q, acc + q, 4);
    }
  }
}

hipError_t launch_guard_fill(uint8_t* ws, const GuardList& g, hipStream_t s) {
  if (g.n <= 0) return hipSuccess;
  if (g.n > kMaxGuards) return hipErrorInvalidValue;
  hipLaunchKernelGGL(guard_fill_kernel, dim3(g.n), dim3(kGuardBytes / 4), 0, s, ws, g);
  return hipGetLastError();
}

hipError_t launch_dump(const DumpCall& c, hipStream_t s) {
  if (c.ws && (c.guards.n > kMaxGuards || !c.bad)) return hipErrorInvalidValue;
  const int64_t per = c.mode == kDumpFold ? 512 : 1024;   // scalars a workgroup
  const int64_t blocks = (c.mode == kDumpCheck ? 0 : (c.n + per - 1) / per) + (c.ws ? 1 : 0);
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
#define CORR_DUMP(T, M)                                                                                           \
  hipLaunchKernelGGL((dump_kernel<T, M>), dim3((unsigned)blocks), dim3(256), 0, s, static_cast<const T*>(c.acc), \
                     c.longrun, c.dst, c.n, c.ws, c.guards, c.bad)
  switch (c.mode) {
    case kDumpCheck: CORR_DUMP(int32_t, kDumpCheck); break;
    case kDumpCopy: CORR_DUMP(int32_t, kDumpCopy); break;   // bits of either type
    case kDumpCopyLong: CORR_DUMP(int32_t, kDumpCopyLong); break;
    case kDumpFold: if (c.is_int) CORR_DUMP(int32_t, kDumpFold); else CORR_DUMP(float, kDumpFold); break;
    case kDumpFoldCopy: if (c.is_int) CORR_DUMP(int32_t, kDumpFoldCopy); else CORR_DUMP(float, kDumpFoldCopy); break;
    case kDumpFoldCopyLong:
      if (c.is_int) CORR_DUMP(int32_t, kDumpFoldCopyLong); else CORR_DUMP(float, kDumpFoldCopyLong);
      break;
    default: return hipErrorInvalidValue;
  }
#undef CORR_DUMP
  return hipGetLastError();
}

}  // namespace corr
