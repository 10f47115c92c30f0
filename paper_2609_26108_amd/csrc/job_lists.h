// Which of several equal lists a job appends to (a returning atomic per list
// instead of one for the whole chip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace chert {

// List of job j among n: every run of n jobs starting at a multiple of n fills
// each list once, so the lists' jobs are as many; the runs are rotated against
// each other by a mixed run number, so that jobs a multiple of n apart -- a
// column of a grid whose width is one -- do not share a list (with j mod n such
// a column's fold directions overran their list's room, and its jobs were
// solved twice).
__host__ __device__ inline int list_of_job(int64_t j, int n) {
  uint32_t r = (uint32_t)(j / n) * 2654435769u;  // 2^32 over the golden ratio
  r ^= r >> 16;
  r *= 2654435769u;
  return (int)((j % n + (r >> 16) % (uint32_t)n) % n);
}

}  // namespace chert
