// Sorting networks over values that one lane holds in registers.  Every index
// is a compile-time constant after unrolling.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pisa {

// The larger of two floats in one instruction without canonicalising the
// operands (the median with +inf); a NaN in `a` loses.
__device__ __forceinline__ float sel_max(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, INFINITY); }

// (values, not references, on both sides of each select)
__device__ __forceinline__ void cx_desc(float& a, float& b) {
  const float x = a, y = b;
  const bool sw = y > x;
  a = sw ? y : x;
  b = sw ? x : y;
}
__device__ __forceinline__ void cx_asc(int& a, int& b) {
  const int x = a, y = b;
  a = min(x, y);
  b = max(x, y);
}
__device__ __forceinline__ void cx_asc(uint64_t& a, uint64_t& b) {
  const uint64_t x = a, y = b;
  const bool sw = y < x;
  a = sw ? y : x;
  b = sw ? x : y;
}

// Batcher's odd-even merge sort of the N = 2^k places LO .. LO + N - 1:
// f(i, j) orders places i < j.  Recursion over templates, so that every place
// is a constant and the values stay in registers.
template <int I, int END, int R, int STEP, typename F>
__device__ __forceinline__ void oddeven_pairs(F& f) {
  if constexpr (I + R < END) {
    f(I, I + R);
    oddeven_pairs<I + STEP, END, R, STEP>(f);
  }
}
template <int LO, int N, int R, typename F>
__device__ __forceinline__ void oddeven_merge(F& f) {
  if constexpr (2 * R < N) {
    oddeven_merge<LO, N, 2 * R>(f);
    oddeven_merge<LO + R, N, 2 * R>(f);
    oddeven_pairs<LO + R, LO + N, R, 2 * R>(f);
  } else {
    f(LO, LO + R);
  }
}
template <int LO, int N, typename F>
__device__ __forceinline__ void oddeven_sort_at(F& f) {
  if constexpr (N > 1) {
    oddeven_sort_at<LO, N / 2>(f);
    oddeven_sort_at<LO + N / 2, N / 2>(f);
    oddeven_merge<LO, N, 1>(f);
  }
}
template <int N, typename F>
__device__ __forceinline__ void oddeven_sort(F&& f) {
  oddeven_sort_at<0, N>(f);
}

template <int K, int N>
__device__ __forceinline__ void bitonic_steps_desc(float (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if ((i & K) == 0) cx_desc(v[i], v[i + K]);
  }
  if constexpr (K > 1) bitonic_steps_desc<K / 2>(v);
}

// Sorts a bitonic sequence of N values, largest first.
template <int N>
__device__ __forceinline__ void bitonic_merge_desc(float (&v)[N]) {
  bitonic_steps_desc<N / 2>(v);
}

template <int N>
__device__ __forceinline__ void sort_desc(float (&v)[N]) {
  oddeven_sort<N>([&](int i, int j) __attribute__((always_inline)) { cx_desc(v[i], v[j]); });
}

// a, b sorted largest first: a becomes the N largest of both, sorted.
template <int N>
__device__ __forceinline__ void merge_top_desc(float (&a)[N], const float (&b)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) a[i] = sel_max(b[N - 1 - i], a[i]);
  bitonic_merge_desc(a);
}

// v[k] for a k that is the same in every lane.  (Recursion: a loop of selects
// is turned into an indexed load, which would put v into scratch memory.)
template <int I, int N>
__device__ __forceinline__ float pick_uniform_at(const float (&v)[N], int k) {
  if constexpr (I + 1 == N) {
    return v[I];
  } else {
    const float x = v[I], rest = pick_uniform_at<I + 1>(v, k);
    return k <= I ? x : rest;
  }
}
template <int N>
__device__ __forceinline__ float pick_uniform(const float (&v)[N], int k) {
  return pick_uniform_at<0>(v, k);
}

}  // namespace pisa
