// Weight rows of a tile's class pairs in LDS.  The classes a tile's box holds
// (few, whatever the cache's class count) get codes whose pairwise sums are
// all different (the marks of a Golomb ruler), so the row of an unordered pair
// is the sum of its codes: with codes stored times the row length, the weight
// of offset o from class p to class q is W[code(p) + code(q) + o] -- one
// addition per edge instead of a product of ids -- and both directions of an
// edge, whose weights are equal, share a row.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace chert {

constexpr int kCodeClasses = 8;    // most classes of a box with staged weights
constexpr int kCodeMaskIds = 64;   // class ids the presence mask covers
// optimal Golomb rulers of 1..8 marks, a mark per byte, lowest first: {0},
// {0 1}, {0 1 3}, {0 1 4 6}, {0 1 4 9 11}, {0 1 4 10 12 17},
// {0 1 4 10 18 23 25}, {0 1 4 9 15 22 32 34}
__constant__ constexpr uint64_t kCodes[kCodeClasses] = {
    0x0ull,          0x100ull,          0x30100ull,          0x6040100ull,
    0xb09040100ull,  0x110c0a040100ull, 0x1917120a040100ull, 0x2220160f09040100ull};
__device__ __forceinline__ int code_of(int nk, int rank) {
  return (int)((kCodes[nk - 1] >> (8 * rank)) & 0xffull);
}

// rows of n classes: the largest sum is twice the last mark
__host__ __device__ inline int code_rows(int n) {
  constexpr int last[kCodeClasses] = {0, 1, 3, 6, 11, 17, 25, 34};
  return 2 * last[n - 1] + 1;
}

// Most classes (at most K) whose rows of n_off weights fit in `bytes`; 0: none.
__host__ inline int code_classes(int K, int n_off, size_t bytes) {
  int n = 0;
  while (n < K && n < kCodeClasses && (size_t)code_rows(n + 1) * n_off * sizeof(double) <= bytes)
    ++n;
  return n;
}

// Stage the weights of the pairs of the classes in `present` (nk of them):
// rows of n_off doubles in W, from the table Wf[K][K][n_off].  All threads.
__device__ __forceinline__ void stage_codes(double* W, const double* Wf, int K, int n_off,
                                            unsigned long long present, int nk) {
  unsigned long long mh = present;
  for (int hi = 0; hi < nk; ++hi, mh &= mh - 1ull) {
    const int kh = __ffsll((long long)mh) - 1;
    unsigned long long ml = present;
    for (int lo = 0; lo <= hi; ++lo, ml &= ml - 1ull) {
      const double* src = Wf + ((int64_t)kh * K + (__ffsll((long long)ml) - 1)) * n_off;
      double* dst = W + (code_of(nk, hi) + code_of(nk, lo)) * n_off;
      for (int o = threadIdx.x; o < n_off; o += blockDim.x) dst[o] = src[o];
    }
  }
}

// code of class id k, times the row length
__device__ __forceinline__ int class_code(unsigned long long present, int nk, int k, int n_off) {
  const int rank = __popcll(present & ((1ull << k) - 1ull));
  return code_of(nk, rank < nk ? rank : nk - 1) * n_off;
}

}  // namespace chert
