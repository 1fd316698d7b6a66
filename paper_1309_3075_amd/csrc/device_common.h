// Device helpers shared by the HIP kernels of the library.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace epochlik {

constexpr int kMaxCategories = 8;
constexpr int kBlock = 256;
constexpr double kLn2 = 0.69314718055994530942;

// Power-of-two rescaling: returns e such that m * 2^-e lies in [0.5, 1) for m > 0
// (0 when m == 0 or not finite).  Exact for any rounding mode.
__device__ inline int scale_exponent(float m) {
  if (!(m > 0.0f) || !isfinite(m)) return 0;
  int e;
  frexpf(m, &e);
  return e;
}
__device__ inline int scale_exponent(double m) {
  if (!(m > 0.0) || !isfinite(m)) return 0;
  int e;
  frexp(m, &e);
  return e;
}
__device__ inline float scale_by_pow2(float x, int e) { return ldexpf(x, -e); }
__device__ inline double scale_by_pow2(double x, int e) { return ldexp(x, -e); }

__device__ inline float dev_exp(float x) { return expf(x); }
__device__ inline double dev_exp(double x) { return exp(x); }
__device__ inline float dev_expm1(float x) { return expm1f(x); }
__device__ inline double dev_expm1(double x) { return expm1(x); }
__device__ inline float dev_cos(float x) { return cosf(x); }
__device__ inline double dev_cos(double x) { return cos(x); }
__device__ inline float dev_sin(float x) { return sinf(x); }
__device__ inline double dev_sin(double x) { return sin(x); }

// Reductions within groups of W consecutive lanes of a 64-wide wavefront.
template <int W, typename T>
__device__ inline T group_max(T v) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) {
    T u = __shfl_xor(v, o, W);
    v = u > v ? u : v;
  }
  return v;
}
template <int W, typename T>
__device__ inline T group_sum(T v) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, W);
  return v;
}

// Deterministic block-wide sum of doubles (fixed tree order), result on thread 0.
template <int NT>
__device__ inline double block_sum(double v, double* smem) {
  const int t = threadIdx.x;
  smem[t] = v;
  __syncthreads();
#pragma unroll
  for (int s = NT / 2; s > 0; s >>= 1) {
    if (t < s) smem[t] += smem[t + s];
    __syncthreads();
  }
  double r = smem[0];
  __syncthreads();
  return r;
}

// Block partial sums of one launch added up inside it.  Every block of the launch (n_blocks of
// them, one slot each) calls this with its sum on thread 0; the last one to arrive sums the slots
// in order (the same order whichever block is last) and writes out[0], and host_out[0] when given.
// A launch of its own for that sum took 1.7-4.8 us plus the gap before it.  `arrived` is 0 before
// the launch and again after it; the slots and the counter go through device-scope atomics, since
// blocks on different XCDs do not share an L2.
template <int NT>
__device__ inline void sum_blocks_in_last(double block_total, double* slots, int slot, int n_blocks,
                                          unsigned* arrived, double* out, double* host_out, double* smem) {
  __shared__ int last;
  if (threadIdx.x == 0) {
    __hip_atomic_store(&slots[slot], block_total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // the slot is written through to device scope before the counter moves; a full release would
    // also write back whatever else the XCD's L2 holds
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const unsigned before = __hip_atomic_fetch_add(arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = before + 1 == (unsigned)n_blocks;
  }
  __syncthreads();
  if (!last) return;
  double acc = 0.0;
  for (int k = threadIdx.x; k < n_blocks; k += NT)
    acc += __hip_atomic_load(&slots[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const double tot = block_sum<NT>(acc, smem);
  if (threadIdx.x == 0) {
    out[0] = tot;
    if (host_out) host_out[0] = tot;
    __hip_atomic_store(arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Barrier of a run between its levels: what its wavefronts exchange is in LDS, so the loads ahead and
// the stores of results stay in flight (a __syncthreads waits for them).
__device__ inline void lds_barrier() {
  __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  __asm__ volatile("" ::: "memory");
}

}  // namespace epochlik
