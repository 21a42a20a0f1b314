// Walks over rows and entries whose end may be the largest int (n and nnz go up
// to 2^31 - 1): a signed index stepped past such an end wraps to a negative one,
// which is below the end again.
#pragma once

#include <hip/hip_runtime.h>

namespace rpk {

// Row behind the last one of the 64-row slice s of n rows (64 s < n).
__host__ __device__ __forceinline__ int slice_end(int n, int s) {
  return n - 64 * s > 64 ? 64 * s + 64 : n;
}

// One lane's share of the entries e0 .. e1 - 1 that a wavefront walks: e0 + lane,
// e0 + lane + 64, ...  Counted from e0 without a sign.
struct LaneEntries {
  int e0;
  unsigned cnt, k;
  __host__ __device__ __forceinline__ LaneEntries(int begin, int end, int lane)
      : e0(begin), cnt((unsigned)(end - begin)), k((unsigned)lane) {}
  __host__ __device__ __forceinline__ bool more() const { return k < cnt; }
  __host__ __device__ __forceinline__ void next() { k += 64u; }
  __host__ __device__ __forceinline__ int at() const { return e0 + (int)k; }
};

// The same for a walk over rows in steps of a workgroup: first < hi and the next
// first of a wavefront, both without a sign (hi at most 2^31 - 1, steps of 1,024 at most).
__host__ __device__ __forceinline__ bool row_below(unsigned first, int hi) { return first < (unsigned)hi; }

}  // namespace rpk
