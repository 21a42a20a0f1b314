// Index and limit arithmetic that host and kernels share.
//
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

// What the certified sum (row_cert) has to know of a row's non-zero entries: the
// exponents of x_j for which every product lies in the exact range of twoprod, from
// the entries' smallest and largest binary exponent (frexp: a = m 2^e, 1/2 <= |m| < 1) as
// 2^(ea + ex - 2) <= |a x| < 2^(ea + ex) has to lie in [2^-968, 2^990), and lsb - 1, lsb
// the exponent of the lowest set bit of any of them.
struct CertLim {
  int xlo, xhi, lsb1;
};

// In a word, for a dictionary row or the range of a slice of rows: 12 bits of lsb - 1,
// ten bits each of the range in steps of four, rounded to the strict side.
__host__ __device__ __forceinline__ int cert_pack(int elo, int ehi, int lsb) {
  const int lo = (-966 - elo + 3) >> 2, hi = (989 - ehi) >> 2;
  return (int)(((unsigned)(hi < 511 ? hi : 511) << 22) | (((unsigned)lo & 0x3ffu) << 12) | ((unsigned)(lsb - 1) & 0xfffu));
}
__host__ __device__ __forceinline__ CertLim cert_unpack(int w) {
  return CertLim{((int)((unsigned)w << 10) >> 22) * 4, (w >> 22) * 4, (int)((unsigned)w << 20) >> 20};
}
// lsb - 1 of a row of the SELL copy in a byte, in steps of 16 rounded down: the test
// has some 48 bits to spare for x_j of like size
__host__ __device__ __forceinline__ signed char cert_pack_lsb(int lsb) { return (signed char)((lsb - 1) >> 4); }
__host__ __device__ __forceinline__ int cert_unpack_lsb(signed char b) { return (int)b * 16; }

}  // namespace rpk
