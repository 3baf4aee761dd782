// One column of a table of partial sums: its rows first, first + 4, ... added in order
// (the rows of one of a workgroup's four waves), sixteen requested at a time.
#pragma once
#include <hip/hip_runtime.h>

namespace sq {

__device__ __forceinline__ float part_rows_sum(const float* __restrict__ col, long long ld, int first, int rows) {
  float sum = 0.f;
  int r = first;
  for (; r + 60 < rows; r += 64) {
    float t[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) t[k] = col[(long long)(r + 4 * k) * ld];
#pragma unroll
    for (int k = 0; k < 16; ++k) sum += t[k];
  }
  if (r < rows) {   // the rest, requested together too: rows past the end read the last one
    float t[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) t[k] = col[(long long)(r + 4 * k < rows ? r + 4 * k : rows - 1) * ld];
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (r + 4 * k < rows) sum += t[k];
  }
  return sum;
}

}  // namespace sq
