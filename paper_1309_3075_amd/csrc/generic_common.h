// Child vectors of the generic kernels: tip state sets and strided dot products.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace epochlik {
namespace {

// The 0/1 indicator of a tip state code (text after Eq. 4): code < K one state,
// K every state (missing), K + 1 + a the caller's ambiguity set a.
__device__ inline uint64_t tip_set(int st, int K, const uint64_t* __restrict__ amb) {
  if (st < K) return 1ull << st;
  if (st == K) return K == 64 ? ~0ull : ((1ull << K) - 1);
  return amb[st - K - 1];
}

// sum_j M[j * stride] * v[j] over j < n, summed in order of j, with the loads of
// up to 16 terms issued together (the matrix entries are mostly not in cache, so
// one load per step would pay the memory latency n times).
template <typename T>
__device__ inline T dot_strided(const T* __restrict__ M, size_t stride, const T* v, int n) {
  T r = 0;
  int j = 0;
  for (; j + 16 <= n; j += 16) {
    T m[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) m[k] = M[(size_t)(j + k) * stride];
#pragma unroll
    for (int k = 0; k < 16; ++k) r += m[k] * v[j + k];
  }
  if (j + 8 <= n) {
    T m[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) m[k] = M[(size_t)(j + k) * stride];
#pragma unroll
    for (int k = 0; k < 8; ++k) r += m[k] * v[j + k];
    j += 8;
  }
  if (j + 4 <= n) {
    T m[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) m[k] = M[(size_t)(j + k) * stride];
#pragma unroll
    for (int k = 0; k < 4; ++k) r += m[k] * v[j + k];
    j += 4;
  }
  for (; j < n; ++j) r += M[(size_t)j * stride] * v[j];
  return r;
}

template <typename T>
__device__ inline T child_vector(int child, int N, int p, int tstride, int K, int Kp, int i, const T* Prow,
                                 const uint8_t* tips, const uint64_t* amb, const T* sL) {
  // (P_child L_child)(i) for a pattern; Prow points at row i of the child's matrix; tstride is the
  // row stride of the tip states (the instance's pattern count).
  if (child < N) {
    const int st = tips[(size_t)child * tstride + p];
    if (st < K) return Prow[st];
    const uint64_t set = tip_set(st, K, amb);
    T r = 0;
    for (int j = 0; j < K; ++j)
      if ((set >> j) & 1) r += Prow[j];
    return r;
  }
  return dot_strided(Prow, 1, sL, K);
}

}  // namespace
}  // namespace epochlik
