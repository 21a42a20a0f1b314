// kernels.h -- gfx950 kernels of the reproducible PBiCGStab hot path.
//
// N > 0 selects the exact arithmetic (FPE of length N + long accumulator, one
// rounding per dot product and per CSR row); N == 0 selects the plain FP64
// comparison path (fma row sums in CSR order, fma dot partials, tree reduction);
// N == LW8 selects the lightweight dot products of Sec. 3.2 (FPEs of length 8
// with early exit, merged with twosum cascades across lanes and workgroups,
// rounded once; bits that do not fit are flagged) with the exact CSR rows.
//
// Row partitioning: the grid has G workgroups; logical block L owns a contiguous
// range of rows.  The hardware hands workgroups to the 8 XCDs round-robin, so
// xcd_block() renumbers them to give each XCD one contiguous eighth of the rows,
// which keeps the SpMV neighbour gathers inside that XCD's L2.
#pragma once
#include <climits>

#include "device.h"
#include "span.h"

namespace rpk {

constexpr int HIST_W = 12;   // doubles per recorded iteration
constexpr int MAX_DOTS = 8;  // reduction slots in the workspace
// Exact cross-lane reduction: each workgroup sums its lanes' FPE components as
// integers in a window of WIN digits of the long-accumulator grid, whose top is
// the highest digit the workgroup's largest component reaches, and adds the
// window into the dot's global long
// accumulator.  Digits that fall below the window (components more than about
// 290 bits below the workgroup's largest) go to the long accumulator directly,
// so nothing is ever dropped.
constexpr int WIN = 12;
// Lightweight mode: FPE length 8; each workgroup publishes a record of LW_REC
// doubles per dot (8 components, the plain tail, the flags as a double).
constexpr int LW8 = 9;
constexpr int LW_N = 8;
constexpr int LW_REC = 10;
// FPE length of the exact row sums (the lightweight mode keeps the exact rows)
template <int N>
constexpr int kRowN = (N == LW8) ? 4 : N;

enum : int { ST_OK = 0, ST_NONFINITE = 5, ST_NOT_CONVERGED = 6, ST_BREAKDOWN = 7 };

// An entry of the row dictionary (Csr::pid): value and 8 (column - row), the
// distance in bytes between the operand's element and the row's own.
// A dictionary row's first entry holds its limits for the certified sum (cert_pack).
struct __align__(16) PatEnt {
  double a;
  int off8, lim;
};
// Dictionary rows are padded with (0, own element) to a multiple of four
// entries, so that a batch reads no entry behind them, and by one more, so that
// different rows lie on different LDS banks.
__host__ __device__ constexpr int pat_stride(int pw) { return ((pw + 3) & ~3) + 1; }
// entries of the LDS set aside for the dictionary in every kernel that multiplies
// by the matrix: 16 KB.  The limit is that reserve, not where the two forms cross: a
// 7-point grid of 128^3 rows takes 19.1 us an SpMV with five values on its diagonal
// (103 different rows), 32.2 from the SELL copy with eight, whose rows do not fit.
constexpr int kPatEntries = 1024;

// Matrix as the kernels see it.  The CSR input is re-laid out at creation as
// SELL-64: slices of 64 consecutive rows (one wavefront), each slice stored
// column-major with the width of its longest row, so that lane l of a wave reads
// entry j of its row at sval[sptr[s] + 64 j + l] -- one coalesced 512-byte load
// per entry index.  Short rows are padded with (value 0, column = own row): the
// exact row sum is unchanged, and a non-finite x[row] already makes the row
// non-finite through its diagonal entry.
struct Csr {
  const long long* sptr;  // [nslices + 1] entry offset of each slice
  const int* scol;        // [sptr[nslices]]
  const double* sval;     // [sptr[nslices]]
  const double* dinv;
  int n;
  // rows first try the certified row sum (decided once per matrix at creation
  // by a probe; every path gives the same bits); with the SELL copy, the limits of
  // slice s are slim[s] (range) and of row i rlsb[i]: a word a row cost 1.0 us of the
  // 32 of an SpMV of 128^3 rows and 14.6M entries
  int cert;
  const int* slim;          // [nslices]
  const signed char* rlsb;  // [64 nslices]
  // slices [0, keep) read their entries with ordinary loads, which leave them
  // in the Infinity Cache for the next SpMV; the rest with non-temporal loads,
  // which leave the cache to the vectors (the same values either way)
  int keep;
  // every dinv_i has the same bits, du (decided at creation): M^-1 is then the
  // scalar du, and a preconditioned vector RN(dinv_i v_i) = RN(du v_i) can be
  // formed where it is read instead of being stored (the same values either way)
  int unif;
  double du;
  // Row dictionary (np > 0): the matrix has few different rows, a row being its
  // list of (column - row, value).  Row r is row pid[r] of the dictionary, whose
  // entry j is pat[pid[r] pat_stride(pw) + j]; swid[s] is the width of slice s,
  // pw the largest.  A kernel copies the dictionary into LDS (pat_load) and reads
  // one byte per row instead of 12 per entry; the SELL copy is then absent.
  const unsigned char* pid;   // [64 nslices]
  const unsigned char* swid;  // [nslices]
  const PatEnt* pat;          // [np pat_stride(pw)]
  int np, pw;
  // Operand window (win > 0): every row's columns lie between wlo before and whi
  // behind it, and scattered, so that one gather of a wavefront touches about as
  // many cache lines as it has lanes.  A workgroup then stages the operand of its
  // rows and the band around them, win doubles, in LDS and gathers there, with
  // 16-bit distances, sdif = column - row + wlo, in place of the columns.
  const unsigned short* sdif;  // [sptr[nslices]]
  int wlo, whi, win;
};

// Device-resident solver state (one per solve, in the caller's workspace).
// resumable: 1 = stopped at maxit with the next iteration's scalars in place,
// 2 = stopped at maxit where the next step breaks down, 0 = otherwise.
struct State {
  double alpha, omega, beta, rho, tau, tau0, tol, true_res;
  double varsigma, zeta;  // pipelined: <r0,s>, <r0,z> of the current iteration (S16, taken in P1)
  double stg;             // deferred reductions: rho after S10 (standard) / beta after S6 (PCG), moved by B / S1
  int iter, maxit, done, status;
  int variant, resumable;
  int lost;     // lightweight mode: dot products that could not keep every bit
  int spmv_go;  // pipelined: 1 when the kernel before an SpMV ran (written by that kernel only)
  int pend;     // deferred reductions: E (PCG: S3) published its dots, A (S10) has not taken them
  int iter_n;   // deferred reductions: iter after the stop test, moved to iter by B (PCG: S1)
};

// Reduction scratch in the caller's workspace (left zeroed after every use).
struct Red {
  double* partials;    // plain mode: [slot][G] workgroup sums
  long long* gsa;      // [copies][MAX_DOTS slots][SA_D] global long accumulators
  int* gflags;         // [slot]
  unsigned* tickets;   // [8] arrival counters; from kSubTickets on, one for each copy (copies > 1)
  int G;               // number of workgroups (or tiles) that publish
  int copies;          // of each accumulator: workgroup b adds into copy b % copies (red_copies)
};
// Additions of many workgroups into one address are performed one after another
// (about 10 ns each), which the end of a kernel waits for: with 512 workgroups
// and one copy of each accumulator, kernel B of a 64^3 solve took 12.8 us, with
// eight 9.1 (128^3: 29.4 and 27.6).  Fewer workgroups queue less, and with few
// copies the threads of a small workgroup load all of them at once (DCAP).
constexpr int kMaxCopies = 8;
constexpr int kSubTickets = 8 + MAX_DOTS;  // behind the counters and the flags
__host__ __device__ constexpr int red_copies(int grid) { return grid >= 256 ? kMaxCopies : grid >= 64 ? 4 : 1; }

// ---------------------------------------------------------------------------
// LDS layout
// ---------------------------------------------------------------------------
// The window of an exact reduction: 64 rows of WIN digits per dot, row l shared
// by lane l of every wavefront.  One digit of padding puts the rows of 16
// consecutive lanes on distinct banks.
constexpr int ROW_STRIDE = WIN + 1;

// room for the row dictionary or the operand window
__host__ __device__ inline size_t pat_bytes(int win) {
  const size_t d = (size_t)kPatEntries * sizeof(PatEnt), w = (((size_t)win + 1) & ~(size_t)1) * 8;
  return w > d ? w : d;
}

__host__ __device__ inline size_t shm_bytes(int N, int K, bool rows, int block, int win = 0) {
  const size_t nw = (size_t)block / 64, k1 = K > 0 ? K : 1;
  const bool exact = N > 0 && N != LW8;
  const size_t sa = exact ? (size_t)K * SA_D * 8 : 0;
  const size_t scat = exact ? (size_t)K * 64 * ROW_STRIDE * 8 : 0;
  const size_t wsa = N > 0 && rows ? nw * SA_D * 8 : 0;
  const size_t wsum = exact ? k1 * WIN * 8 : N == LW8 ? nw * k1 * LW_REC * 8 : 0;
  const size_t pat = rows ? pat_bytes(win) : 0;
  return pat + sa + scat + wsa + wsum + 16 * 8 + MAX_DOTS * 4 + MAX_DOTS * 8 + MAX_DOTS * 4 + (4 + MAX_DOTS) * 4;
}

template <int N>
struct Shm {
  PatEnt* pat;      // row dictionary of the matrix or operand window (kernels with rows)
  long long* sa;    // K * SA_D    long accumulators (rare path)
  long long* scat;  // K * 64 * ROW_STRIDE window rows
  long long* wsa;   // nw * SA_D   row fallback accumulators (kernels with rows)
  long long* wsum;  // K * WIN     window sums (lightweight: nw * K * LW_REC doubles)
  double* pbuf;     // 16          plain per-wave sums
  int* imax;        // MAX_DOTS    highest digit of the workgroup's components, -1: none
  double* res;      // MAX_DOTS
  int* flag;        // MAX_DOTS
  int* misc;        // 4 + MAX_DOTS  ([1..K] flags, [10] last-arrival, [11] sink)
};

template <int N>
__device__ __forceinline__ Shm<N> shm_carve(char* base, int K, bool rows, int win = 0) {
  Shm<N> s;
  const size_t nw = blockDim.x / 64, k1 = K > 0 ? K : 1;
  constexpr bool exact = N > 0 && N != LW8;
  size_t off = 0;
  s.pat = (PatEnt*)(base + off);
  off += rows ? pat_bytes(win) : 0;
  s.sa = (long long*)(base + off);
  off += exact ? (size_t)K * SA_D * 8 : 0;
  s.scat = (long long*)(base + off);
  off += exact ? (size_t)K * 64 * ROW_STRIDE * 8 : 0;
  s.wsa = (long long*)(base + off);
  off += N > 0 && rows ? nw * SA_D * 8 : 0;
  s.wsum = (long long*)(base + off);
  off += exact ? k1 * WIN * 8 : N == LW8 ? nw * k1 * LW_REC * 8 : 0;
  s.pbuf = (double*)(base + off);
  off += 16 * 8;
  s.imax = (int*)(base + off);
  off += MAX_DOTS * 4;
  s.res = (double*)(base + off);
  off += MAX_DOTS * 8;
  s.flag = (int*)(base + off);
  off += MAX_DOTS * 4;
  s.misc = (int*)(base + off);
  return s;
}

// Copy A's row dictionary into LDS (nothing where it has none); a barrier must
// follow before any row is computed.
template <int N>
__device__ __forceinline__ void pat_load(const Csr& A, const Shm<N>& s) {
  const int cnt = A.np * pat_stride(A.pw);
  for (int k = threadIdx.x; k < cnt; k += blockDim.x) ((int4*)s.pat)[k] = ((const int4*)A.pat)[k];
}

// zero the K long accumulators, window rows and flags of this block (must precede any deposit)
template <int N>
__device__ __forceinline__ void shm_init(const Shm<N>& s, int K) {
  if (N > 0 && N != LW8) {
    for (int k = threadIdx.x; k < K * SA_D; k += blockDim.x) s.sa[k] = 0;
    for (int k = threadIdx.x; k < K * 64 * ROW_STRIDE; k += blockDim.x) s.scat[k] = 0;
  }
  if (threadIdx.x < MAX_DOTS) {
    s.flag[threadIdx.x] = 0;
    s.imax[threadIdx.x] = -1;
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Partitioning
// ---------------------------------------------------------------------------
__device__ __forceinline__ int xcd_block(int b, int G) {
  const int G8 = G & ~7;
  if (b >= G8) return b;
  return (b & 7) * (G8 >> 3) + (b >> 3);
}

struct Range {
  int lo, hi;
};

// contiguous row range of logical block L out of G (chunk rounded to 64 rows)
__device__ __forceinline__ Range block_rows(int n, int L, int G) {
  long long chunk = ((long long)n + G - 1) / G;
  chunk = (chunk + 63) & ~63ll;
  long long lo = (long long)L * chunk, hi = lo + chunk;
  if (lo > n) lo = n;
  if (hi > n) hi = n;
  return Range{(int)lo, (int)hi};
}

// ---------------------------------------------------------------------------
// Dot accumulators
// ---------------------------------------------------------------------------
template <int N>
struct Dot {
  Fpe<N> f;
  __device__ __forceinline__ void zero() { fpe_zero(f); }
  __device__ __forceinline__ void add(double a, double b, long long* sa, int* flag) {
    acc_prod(f, a, b, sa, flag);
  }
};

template <>
struct Dot<0> {
  double s;
  __device__ __forceinline__ void zero() { s = 0.0; }
  __device__ __forceinline__ void add(double a, double b, long long*, int*) { s = fma(a, b, s); }
};

// Lightweight accumulator (Sec. 3.2): an FPE of 8 doubles with early exit and
// nothing behind it.  What the FPE cannot hold (a cascade that still carries an
// error after the last component, or a product outside the range where twoprod
// is exact) is added to a plain FP64 tail and flagged F_LOST: the result is then
// accurate but no longer guaranteed to be correctly rounded or reproducible.
// When nothing is lost, the FPE holds the exact sum and its rounding equals the
// exact dot product bit for bit.
template <>
struct Dot<LW8> {
  Fpe<LW_N> f;
  double tail;
  int fl;
  __device__ __forceinline__ void zero() {
    fpe_zero(f);
    tail = 0.0;
    fl = 0;
  }
  // insert one double (all lanes of the wavefront call it together)
  __device__ __forceinline__ void put(double x) {
    const double l = fpe_add_w<LW_N, 0>(f, x);
    if (l != 0.0) {
      tail += l;
      fl |= F_LOST;
    }
  }
  __device__ __forceinline__ void add(double a, double b, long long*, int*) {
    const double p = a * b;
    const double ap = fabs(p);
    const bool ok = ap >= kProdLo && ap < kProdHi;
    const double e = ok ? fma(a, b, -p) : 0.0;
    const double l1 = fpe_add_w<LW_N, 0>(f, ok ? p : 0.0);
    const double l2 = fpe_add_w<LW_N, 1>(f, e);
    const bool extreme = !ok && !(p == 0.0 && (a == 0.0 || b == 0.0));
    if (l1 != 0.0 || l2 != 0.0 || extreme) {
      if (!isfinite(a) || !isfinite(b)) {
        fl |= F_NONFINITE;
      } else {
        tail += l1;
        tail += l2;
        if (extreme) tail = fma(a, b, tail);
        fl |= F_LOST;
      }
    }
  }
  // absorb another accumulator's record (components largest first)
  __device__ __forceinline__ void absorb(const double (&c)[LW_N], double t, int f2) {
#pragma unroll
    for (int k = 0; k < LW_N; ++k) put(c[k]);
    tail += t;
    fl |= f2;
  }
  // merge over the lanes of the wavefront whose index differs below `width`
  // (a power of two <= 64); lane 0 ends with the merged value of lanes 0..width-1
  __device__ __forceinline__ void wave_merge(int width) {
#pragma unroll 1
    for (int off = 1; off < width; off <<= 1) {  // kept rolled: the body is large
      double c[LW_N];
#pragma unroll
      for (int k = 0; k < LW_N; ++k) c[k] = __shfl_xor(f.c[k], off, 64);
      const double t = __shfl_xor(tail, off, 64);
      const int f2 = __shfl_xor(fl, off, 64);
      absorb(c, t, f2);
    }
  }
};

// ---------------------------------------------------------------------------
// CSR rows
// ---------------------------------------------------------------------------
// Gathers: the value the SpMV multiplies a_ij by, in two parts: the memory
// access, by column (load) or by a 32-bit byte offset (load8), and fin(v),
// arithmetic on the loaded value.  The row loops issue the loads of a batch of
// entries first and apply fin afterwards, so that no load waits for the one
// before it.
// Raw is what the access gives; kDict marks gathers used with a row dictionary
// only.
struct GatherX {  // plain vector
  using Raw = double;
  static constexpr bool kDict = false;
  const double* __restrict__ x;
  __device__ __forceinline__ double load(int c) const { return x[c]; }
  __device__ __forceinline__ double load8(unsigned o) const { return *(const double*)((const char*)x + o); }
  __device__ __forceinline__ double fin(double v) const { return v; }
};
// M^-1 v for a uniform Jacobi vector (Csr::unif), formed at the gather:
// RN(du * v_c), the value a stored copy would hold.
struct GatherScaled {
  using Raw = double;
  static constexpr bool kDict = false;
  double du;
  const double* __restrict__ v;
  __device__ __forceinline__ double load(int c) const { return v[c]; }
  __device__ __forceinline__ double load8(unsigned o) const { return *(const double*)((const char*)v + o); }
  __device__ __forceinline__ double fin(double x) const { return du * x; }
};

// M^-1 of a vector that is itself an update of others, formed at the gather (a
// uniform Jacobi vector and a row dictionary): S4 + S5, q = fma(-alpha, s, r) ...
struct GatherQ {
  struct Raw {
    double s, r;
  };
  static constexpr bool kDict = true;
  double du, alpha;
  const double *__restrict__ s, *__restrict__ r;
  __device__ __forceinline__ Raw load8(unsigned o) const {
    return Raw{*(const double*)((const char*)s + o), *(const double*)((const char*)r + o)};
  }
  __device__ __forceinline__ double own(Raw v) const { return fma(-alpha, v.s, v.r); }
  __device__ __forceinline__ double fin(Raw v) const { return du * own(v); }
};
// ... and S12 + S1, p = fma(beta, fma(-omega, s, p), r)
struct GatherP {
  struct Raw {
    double p, s, r;
  };
  static constexpr bool kDict = true;
  double du, beta, omega;
  const double *__restrict__ p, *__restrict__ s, *__restrict__ r;
  __device__ __forceinline__ Raw load8(unsigned o) const {
    return Raw{*(const double*)((const char*)p + o), *(const double*)((const char*)s + o),
               *(const double*)((const char*)r + o)};
  }
  __device__ __forceinline__ double own(Raw v) const { return fma(beta, fma(-omega, v.s, v.p), v.r); }
  __device__ __forceinline__ double fin(Raw v) const { return du * own(v); }
};

// A matrix entry or column index: non-temporal (NT) or ordinary load.
template <bool NT, class T>
__device__ __forceinline__ T ld_entry(const T* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}

// Where a wavefront finds the entries of its 64 rows.  batch() gives this lane's
// entries j0..j0+B-1 as values a and gathered operands b: all value / column
// loads, then all gathers, so that a lane keeps many independent loads in
// flight; the width w is uniform over the wavefront, and slots from w on have
// the value 0 and an operand of this row.  at(l, j, ..) gives entry j < w of
// lane l's row.
template <bool NT>
struct SellSrc {  // the SELL-64 copy: sv, sc at entry 0 of the slice's first row
  const double* sv;
  const int* sc;
  template <int B, class Gth>
  __device__ __forceinline__ void batch(const Gth& gx, int j0, int w, double (&a)[B], double (&b)[B]) const {
    const unsigned lane = threadIdx.x & 63;
    int c[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const size_t j = (size_t)(j0 + u < w ? j0 + u : w - 1) * 64;
      a[u] = ld_entry<NT>((const double*)((const char*)(sv + j) + lane * 8u));
      c[u] = ld_entry<NT>((const int*)((const char*)(sc + j) + lane * 4u));
    }
#pragma unroll
    for (int u = 0; u < B; ++u) b[u] = gx.load(c[u]);
#pragma unroll
    for (int u = 0; u < B; ++u) {
      b[u] = gx.fin(b[u]);
      if (j0 + u >= w) a[u] = 0.0;
    }
  }
  template <class Gth>
  __device__ __forceinline__ void at(const Gth& gx, int l, int j, double& a, double& b) const {
    a = sv[(size_t)j * 64 + l];
    b = gx.fin(gx.load(sc[(size_t)j * 64 + l]));
  }
};
struct PatSrc {  // the row dictionary (Csr::pid) in LDS
  const PatEnt* pat;
  unsigned row8;  // byte offset of this lane's row (at most n - 1)
  int at0;        // first entry of its dictionary row
  template <int B, class Gth>
  __device__ __forceinline__ void batch(const Gth& gx, int j0, int w, double (&a)[B], double (&b)[B]) const {
    (void)w;
    const PatEnt* e = pat + at0 + j0;
    unsigned o[B];
    typename Gth::Raw v[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      a[u] = e[u].a;
      o[u] = row8 + (unsigned)e[u].off8;
    }
#pragma unroll
    for (int u = 0; u < B; ++u) v[u] = gx.load8(o[u]);
#pragma unroll
    for (int u = 0; u < B; ++u) b[u] = gx.fin(v[u]);
  }
  template <class Gth>
  __device__ __forceinline__ void at(const Gth& gx, int l, int j, double& a, double& b) const {
    const PatEnt* e = pat + __builtin_amdgcn_readlane(at0, l) + j;
    a = e->a;
    b = gx.fin(gx.load8((unsigned)__builtin_amdgcn_readlane((int)row8, l) + (unsigned)e->off8));
  }
};
template <bool NT>
struct WinSrc {  // the SELL-64 copy with the operand window: w0 at the wavefront's first row, wlo before
  const double* sv;
  const unsigned short* sd;
  const double* w0;
  template <int B, class Gth>
  __device__ __forceinline__ void batch(const Gth&, int j0, int w, double (&a)[B], double (&b)[B]) const {
    const unsigned lane = threadIdx.x & 63;
    unsigned c[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const size_t j = (size_t)(j0 + u < w ? j0 + u : w - 1) * 64;
      a[u] = ld_entry<NT>((const double*)((const char*)(sv + j) + lane * 8u));
      c[u] = ld_entry<NT>((const unsigned short*)((const char*)(sd + j) + lane * 2u));
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
      b[u] = w0[lane + c[u]];
      if (j0 + u >= w) a[u] = 0.0;
    }
  }
  template <class Gth>
  __device__ __forceinline__ void at(const Gth&, int l, int j, double& a, double& b) const {
    a = sv[(size_t)j * 64 + l];
    b = w0[l + sd[(size_t)j * 64 + l]];
  }
};

// Stage the operand window of rows R (Csr::win): gathered and finished once an
// element, zero outside the matrix.  Four loads in flight a thread.  Ends with a
// barrier.
template <int N, class Gth>
__device__ __forceinline__ void win_load(const Csr& A, const Gth& gx, Range R, const Shm<N>& s) {
  double* win = (double*)s.pat;
  const int n = R.hi > R.lo ? R.hi - R.lo + A.wlo + A.whi : 0;
  const int c0 = R.lo - A.wlo;
  for (int k0 = threadIdx.x; k0 < n; k0 += 4 * blockDim.x) {
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + k0 + u * (int)blockDim.x;
      v[u] = gx.load(c < 0 ? 0 : c < A.n ? c : A.n - 1);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = k0 + u * (int)blockDim.x, c = c0 + k;
      if (k < n) win[k] = c >= 0 && c < A.n ? gx.fin(v[u]) : 0.0;
    }
  }
  // rows of the last slice behind R
  for (int k = n + threadIdx.x; k < A.win; k += blockDim.x) win[k] = 0.0;
  __syncthreads();
}

// Exact fast path of one row in one lane: FPE of the twoprod terms of entries
// j = 0..w-1.  Sets `bad` when the FPE overflows or a product needs the
// integer path.
template <int N, class Src, class Gth>
__device__ __forceinline__ double row_fast(const Src& src, const Gth& gx, int w, bool& bad) {
  Fpe<N> f;
  fpe_zero(f);
  bool ovf = false;
  for (int j0 = 0; j0 < w; j0 += 4) {
    double a[4], b[4];
    src.template batch<4>(gx, j0, w, a, b);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double p = a[u] * b[u];
      const double ap = fabs(p);
      // no per-lane branch: an out-of-range product inserts 0 and flags the row
      const bool okp = ap >= kProdLo && ap < kProdHi;
      const double e = okp ? fma(a[u], b[u], -p) : 0.0;
      const double l1 = fpe_add_w<N, 0>(f, okp ? p : 0.0);
      const double l2 = fpe_add_w<N, (N > 1 ? 1 : 0)>(f, e);
      ovf |= (l1 != 0.0) | (l2 != 0.0) | (!okp && !(p == 0.0 && (a[u] == 0.0 || b[u] == 0.0)));
    }
  }
  bad = ovf;
  return ovf ? 0.0 : fpe_round(f);
}

// twosum as a value (r = RN(x + y)) and its exact error in `err`
__device__ __forceinline__ double tsum(double x, double y, double& err) {
  const double r = x + y;
  const double z = r - x;
  err = (x - (r - z)) + (y - z);
  return r;
}

// Certified fast path of one row in one lane: the compensated dot product of
// Ogita, Rump and Oishi (2005, Dot2) with its error bound, summed pairwise.
// With p_j + e_j = a_j x_j (twoprod, exact for products in range), each batch
// of eight products is added by a tree of twosums (exact) and the batch sum
// into the running sum s by one more; with t the errors of those eight
// additions, the row sum is exactly T = s + sum(t + e), sixteen terms per
// batch.  q = fl(sum(t + e)), also summed pairwise, is within
// E = gamma_k * sum(|t| + |e|) of that sum for any order of the additions
// (k at least the number of terms).  With (y, r) = twosum(s, q), T = y + r + d
// with |d| <= E, so y = RN(T) whenever |r| + E is below half the gap from y to
// its neighbours.  No bound can settle a T that is a rounding midpoint itself,
// and sums of a few short products often are (a quarter of the 7-point rows);
// there the additions into q are usually exact, because all their operands are
// multiples of one power of two: a_j is an odd multiple of at least 2^lsb (the
// row's smallest), x_j a multiple of 2^(ex_j - 53) with
// ex_j its binary exponent, so every p, e and t, and every partial sum of them,
// is a multiple of U = 2^(lsb + min ex - 53).  A partial sum is at most
// m = sum(|t| + |e|) in magnitude; where m < 2^52 U (the computed m is within
// 2^-40 of it), it is below 2^53 U and hence a double: q is the exact sum, T =
// s + q, and y = RN(s + q) = RN(T) whatever it is.  The products are in range
// by the same exponents (CertLim), which costs three integer operations
// an entry instead of four comparisons; an x_j = 0 counts as exponent 0, which
// can only make the tests stricter (it takes the exactness test from rows that hold
// zeros beside values above some 2^48; leaving zeros out costs two operations an entry,
// 76 -> 81 us of the 27-point 159^3 SpMV).  lsb and the exponents are those of the row
// (the exponents, in the SELL copy, of its slice): one entry of many bits in a matrix of
// short ones (0.1 on a boundary row) then leaves the other rows certified, where with
// limits of the whole matrix it left none.  Returns false -- the caller then takes the
// FPE path -- when neither shows it, or for a product out of range or a sum that
// is non-finite or, for the bound, zero, tiny or huge.  When it returns true, y
// is the correctly rounded row sum: the same bits as the FPE path.  Checking
// every addition into q for exactness by a twosum instead cost 105 more
// operations a row: with it the kernels B and D of the 128^3 standard loop took
// 34.9 and 40.2 us, with the exponents 27.2 and 32.5 (the 27-point 159^3 SpMV 127
// and 81).
struct CertSum {
  double s = 0.0, q = 0.0, m = 0.0;
  int elo = INT_MAX, ehi = INT_MIN;  // binary exponents of the x_j
};

// A row's limits as they are held.
struct PatLim {
  const PatEnt* row;  // its first entry, read again when the sums are there
  __device__ __forceinline__ CertLim get() const { return cert_unpack(row->lim); }
};
// Both words are read at the start of a row: read behind the entries' addresses, the
// gathers of an SpMV of 400,000 rows with 15 random columns took 39.0 us, so 36.0.
struct SellLim {
  int range;
  signed char lsb;
  __device__ __forceinline__ SellLim(const Csr& A, int sl, int i) : range(A.slim[sl]), lsb(A.rlsb[i]) {}
  __device__ __forceinline__ CertLim get() const {
    CertLim l = cert_unpack(range);
    l.lsb1 = cert_unpack_lsb(lsb);
    return l;
  }
};

// Whether the sums prove y = RN(T) (terms: entries summed, padding included).
__device__ __forceinline__ bool cert_finish(const CertLim& lim, const CertSum& c, int terms, double& y) {
  const double s = c.s, q = c.q, m = c.m;
  y = s + (q + 0.0);  // +0 where both are zero
  const double ay = fabs(y);
  const bool in = c.elo >= lim.xlo && c.ehi <= lim.xhi && ay < 0x1p1020;  // false for a NaN y
  // every error term is 0 (the sum is s exactly, +0 for a zero row), or every
  // addition into q was exact
  const bool exactq = m == 0.0 || __builtin_amdgcn_frexp_exp(m) <= c.elo + lim.lsb1;
  const double k = 2.0 * terms + 2.0;  // two error terms per entry
  const double E = (m * (k * 0x1p-53)) * (1.0 + 0x1p-28) + k * 0x1p-1074;
  const double z = y - s;
  const double r = (s - (y - z)) + (q - z);
  // the gap below |y|, the smaller one
  const double gap = ay - __longlong_as_double(__double_as_longlong(ay) - 1ll);
  const bool bound = ay >= 0x1p-960 && (fabs(r) + E) * (2.0 + 0x1p-49) < gap;
  return in && (exactq || bound);
}

template <int B, class Src, class Gth>
__device__ __forceinline__ void cert_batch(const Src& src, const Gth& gx, int j0, int w, CertSum& c) {
  double a[B], b[B];
  src.template batch<B>(gx, j0, w, a, b);
#pragma unroll
  for (int i = 0; i < B; i += 2) {
    const int e0 = __builtin_amdgcn_frexp_exp(b[i]), e1 = __builtin_amdgcn_frexp_exp(b[i + 1]);
    c.elo = min(c.elo, min(e0, e1));
    c.ehi = max(c.ehi, max(e0, e1));
  }
  double p[B], r[B], q[B / 2], m[B / 2];
#pragma unroll
  for (int u = 0; u < B; ++u) {
    p[u] = a[u] * b[u];
    r[u] = fma(a[u], b[u], -p[u]);
  }
  // pairs are added as soon as their operands exist, which keeps the live
  // values of a batch few
#pragma unroll
  for (int i = 0; i < B / 2; ++i) {
    double t;
    const double s = tsum(p[2 * i], p[2 * i + 1], t);
    q[i] = (r[2 * i] + r[2 * i + 1]) + t;
    m[i] = (fabs(r[2 * i]) + fabs(r[2 * i + 1])) + fabs(t);
    p[i] = s;
  }
#pragma unroll
  for (int width = B / 4; width >= 1; width >>= 1)
#pragma unroll
    for (int i = 0; i < width; ++i) {
      double t;
      p[i] = tsum(p[2 * i], p[2 * i + 1], t);
      q[i] = (q[2 * i] + q[2 * i + 1]) + t;
      m[i] = (m[2 * i] + m[2 * i + 1]) + fabs(t);
    }
  if (j0 == 0) {
    c.s = p[0];
    c.q = q[0];
    c.m = m[0];
  } else {
    double t;
    c.s = tsum(c.s, p[0], t);
    c.q += q[0] + t;
    c.m += m[0] + fabs(t);
  }
}

template <class Lim, class Src, class Gth>
__device__ __forceinline__ bool row_cert(const Lim& lim, const Src& src, const Gth& gx, int w, double& y) {
  CertSum c;
  int j0 = 0;
  for (; w - j0 > 4; j0 += 8) cert_batch<8>(src, gx, j0, w, c);
  if (j0 < w) {  // a remainder of up to four entries
    cert_batch<4>(src, gx, j0, w, c);
    j0 += 4;
  }
  return cert_finish(lim.get(), c, j0, y);
}

// Exact slow path: the whole wavefront sums lane l's row in its private long
// accumulator through exact integer products; lane 0 rounds it.
template <class Src, class Gth>
__device__ inline double row_slow(const Src& src, int l, const Gth& gx, int w, long long* wsa) {
  const int lane = threadIdx.x & 63;
  for (int k = lane; k < SA_D; k += 64) wsa[k] = 0;
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_wave_barrier();
  bool nf = false;
  for (int j = lane; j < w; j += 64) {
    double a, b;
    src.at(gx, l, j, a, b);
    if (!isfinite(a) || !isfinite(b)) nf = true;
    else sa_add_prod(wsa, a, b);
  }
  const bool any_nf = __ballot(nf) != 0ull;
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_wave_barrier();
  // with the digits one a lane: in lane 0 alone, the SpMV of 100^3 rows of wide
  // exponents took 1,225 us, 514 so
  double r = sa_round(wsa);
  if (any_nf) r = __longlong_as_double(0x7ff8000000000000ll);
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_wave_barrier();
  return r;
}

// Plain rows: a chain of fmas in entry order.
template <class Src, class Gth>
__device__ __forceinline__ double row_plain(const Src& src, const Gth& gx, int w) {
  double acc = 0.0;
  int j0 = 0;
  for (; w - j0 > 4; j0 += 8) {
    double a[8], b[8];
    src.template batch<8>(gx, j0, w, a, b);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (j0 + u < w) acc = fma(a[u], b[u], acc);
  }
  if (j0 < w) {
    double a[4], b[4];
    src.template batch<4>(gx, j0, w, a, b);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (j0 + u < w) acc = fma(a[u], b[u], acc);
  }
  return acc;
}

// Exact rows of a wavefront without the certificate: the FPE, then the integer
// path for the rows that need it.
template <int N, class Src, class Gth>
__device__ __forceinline__ double rows_fpe(const Src& src, const Gth& gx, int w, bool valid, long long* wsa_block) {
  bool bad = false;
  double y = row_fast<kRowN<N>>(src, gx, w, bad);
  bad = bad && valid;
  unsigned long long m = __ballot(bad);
  if (m) {
    long long* wsa = wsa_block + (size_t)(threadIdx.x >> 6) * SA_D;
    while (m) {
      const int l = __ffsll((long long)m) - 1;
      m &= m - 1ull;
      const double val = row_slow(src, l, gx, w, wsa);
      if ((int)(threadIdx.x & 63) == l) y = val;
    }
  }
  return y;
}

// This workgroup's rows R (R.lo a multiple of 64), one a thread at a time:
// pre(i) loads what the kernel needs of its own row i (called for rows of R
// only), use(i, ok, v, p) takes the row value v = (A g)_i and p = pre(i).  The
// entries come from the row dictionary where the matrix has one, else from the
// SELL copy, whose slice decides the kind of load (Csr::keep).  Exact rows try
// the certified compensated sum first where the matrix's probe chose it: its
// dependency chain is a few additions per entry, an FPE insertion's several
// twosums with a data-dependent exit after each; a wavefront with a row that is
// not certified takes all its rows the other way (its entries are in the caches
// by then).  Every path gives the same values.  With the dictionary the loop is
// bound by vector issue and by the L1's line lookups together, of which a gather of
// 64 lanes takes about 17: busy in the 27-point 159^3 SpMV 70 % and 81 % of the time
// (plain rows 26 % and all of it), in D3 at 128^3 52 % and 56 % (19 % and 76 %).
// Loading the next row's id, operands and own values ahead of this row's sums was
// slower (D 32.9 instead of 27.4 us at 128^3), and so was a second pass for the rows
// that are not certified.
// Win: the operand comes from LDS (Csr::win).
template <int N, bool Win = false, class Gth, class Pre, class Use>
__device__ __forceinline__ void for_rows(const Csr& A, const Gth& gx, Range R, const Shm<N>& s, Pre pre, Use use) {
  if constexpr (Win) win_load(A, gx, R, s);
  // the wavefront's 64 rows (one slice)
  for (unsigned at = __builtin_amdgcn_readfirstlane(R.lo + (int)(threadIdx.x & ~63u)); row_below(at, R.hi);
       at += blockDim.x) {
    const int first = (int)at, i = first + (int)(threadIdx.x & 63), sl = first >> 6;
    const bool ok = i < R.hi;
    double y = 0.0;
    if constexpr (Win) {
      const long long off = A.sptr[sl];
      const int w = (int)((A.sptr[sl + 1] - off) >> 6);
      const double* w0 = (const double*)s.pat + (first - R.lo);
      const WinSrc<false> kept{A.sval + off, A.sdif + off, w0};
      const WinSrc<true> passing{A.sval + off, A.sdif + off, w0};
      const SellLim lim(A, sl, i);
      const auto p = pre(ok ? i : R.hi - 1);
      if constexpr (N == 0) {
        y = sl < A.keep ? row_plain(kept, gx, w) : row_plain(passing, gx, w);
      } else {
        const bool cert = A.cert && (sl < A.keep ? row_cert(lim, kept, gx, w, y) : row_cert(lim, passing, gx, w, y));
        if (__ballot(ok && !cert) != 0ull) y = rows_fpe<N>(kept, gx, w, ok, s.wsa);
      }
      use(i, ok, y, p);
    } else if (Gth::kDict || A.np) {
      const int w = __builtin_amdgcn_readfirstlane((int)A.swid[sl]);
      const PatSrc src{s.pat, (unsigned)(i < A.n ? i : A.n - 1) * 8u, (int)A.pid[i] * pat_stride(A.pw)};
      const auto p = pre(ok ? i : R.hi - 1);
      if constexpr (N == 0) {
        y = row_plain(src, gx, w);
      } else {
        const bool cert = A.cert && row_cert(PatLim{s.pat + src.at0}, src, gx, w, y);
        if (__ballot(ok && !cert) != 0ull) y = rows_fpe<N>(src, gx, w, ok, s.wsa);
      }
      use(i, ok, y, p);
    } else if constexpr (!Gth::kDict) {
      const long long off = A.sptr[sl];
      const int w = (int)((A.sptr[sl + 1] - off) >> 6);
      const SellSrc<false> kept{A.sval + off, A.scol + off};
      const SellSrc<true> passing{A.sval + off, A.scol + off};
      const SellLim lim(A, sl, i);
      const auto p = pre(ok ? i : R.hi - 1);
      if constexpr (N == 0) {
        y = sl < A.keep ? row_plain(kept, gx, w) : row_plain(passing, gx, w);
      } else {
        const bool cert = A.cert && (sl < A.keep ? row_cert(lim, kept, gx, w, y) : row_cert(lim, passing, gx, w, y));
        if (__ballot(ok && !cert) != 0ull) y = rows_fpe<N>(kept, gx, w, ok, s.wsa);
      }
      use(i, ok, y, p);
    }
  }
}

// (A M^-1 v): gathers the stored preconditioned vector vh, or, for a uniform
// Jacobi vector (Unif), v itself scaled at the gather (same values)
template <int N, bool Unif, bool Win = false, class Pre, class Use>
__device__ __forceinline__ void for_rows_hat(const Csr& A, const double* __restrict__ v, const double* __restrict__ vh,
                                             Range R, const Shm<N>& s, Pre pre, Use use) {
  if constexpr (Unif) for_rows<N, Win>(A, GatherScaled{A.du, v}, R, s, pre, use);
  else for_rows<N, Win>(A, GatherX{vh}, R, s, pre, use);
}

// ---------------------------------------------------------------------------
// Exact workgroup reduction of one dot product into a window record
// ---------------------------------------------------------------------------
__device__ __forceinline__ int wave_max_int(int v) {
  // DPP within rows of 16 lanes (shifts 1, 2, 3, then 4 and 8 on the upper
  // banks), then the row broadcasts of lanes 15 and 31: lane 63 ends with the
  // maximum.  Lanes a step does not write keep INT_MIN, which max ignores.
  constexpr int lo = -2147483647 - 1;
  v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x111, 0xf, 0xf, false));  // row_shr:1
  v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x112, 0xf, 0xf, false));  // row_shr:2
  v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x113, 0xf, 0xf, false));  // row_shr:3
  v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x114, 0xf, 0xe, false));  // row_shr:4
  v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x118, 0xf, 0xc, false));  // row_shr:8
  v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x142, 0xa, 0xf, false));  // row_bcast:15
  v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x143, 0xc, 0xf, false));  // row_bcast:31
  return __builtin_amdgcn_readlane(v, 63);
}

// Sum of v over the wavefront, in lane 63: DPP within rows of 16 lanes, then the
// row broadcasts of lanes 15 and 31 (lanes a step does not write add 0).
__device__ __forceinline__ long long wave_sum_i64(long long v) {
#define RPK_STEP(ctrl, rows)                                                                          \
  {                                                                                                   \
    const int lo = __builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xf, false);                    \
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), ctrl, rows, 0xf, false);            \
    v += (long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);                        \
  }
  RPK_STEP(0x111, 0xf)  // row_shr:1
  RPK_STEP(0x112, 0xf)  // row_shr:2
  RPK_STEP(0x114, 0xf)  // row_shr:4
  RPK_STEP(0x118, 0xf)  // row_shr:8
  RPK_STEP(0x142, 0xa)  // row_bcast:15
  RPK_STEP(0x143, 0xc)  // row_bcast:31
#undef RPK_STEP
  return v;
}

// The highest grid digit that digits3 gives a non-zero value for any double of
// magnitude at most |c| (c != 0).
__device__ __forceinline__ int digits3_top(double c) {
  const int ex = (int)(((unsigned long long)__double_as_longlong(c) >> 52) & 0x7ffull);
  return (((ex > 1 ? ex : 1) - 1075 - SA_LSB) >> 5) + 2;
}

// This lane's FPE into its window row (digit 0 = grid digit d0; d0 + WIN - 1 is
// at or above every component's top digit; digits below d0 go to the long
// accumulator `sa`): the digits3 values of each component, by LDS atomics, as
// lane l of every wavefront shares row l.
template <int N>
__device__ __forceinline__ void lane_deposit(const Fpe<N>& f, int d0, long long* row, long long* sa, int* flag) {
  bool below = false;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    long long D[3];
    int idx = digits3(f.c[k], D) - d0;
    if (f.c[k] == 0.0) idx = 0;  // three zeros, added anywhere in the row
    if (idx >= 0) {
#pragma unroll
      for (int j = 0; j < 3; ++j) lds_add(row + idx + j, D[j]);
    } else {
      below = true;
    }
  }
  if (__builtin_expect(below, 0)) {  // rare: components whose low digits lie below the window
#pragma unroll
    for (int k = 0; k < N; ++k) {
      long long D[3];
      const int dg = digits3(f.c[k], D);
      if (f.c[k] == 0.0 || dg >= d0) continue;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        if (dg + j >= d0) {
          lds_add(row + (dg + j - d0), D[j]);
        } else if (D[j] != 0) {
          lds_add(sa + dg + j, D[j]);
          atomicOr(flag, F_SA);
        }
      }
    }
  }
}

// The K dots of the workgroup as windows: dot j's sum is that of the digits
// s.wsum[j WIN + k] at grid digits s.imax[j] - (WIN - 1) + k (nothing where
// s.imax[j] < 0) and of the long accumulator s.sa + j SA_D where s.flag[j] says
// F_SA.  Every thread calls it, after shm_init; ends with a barrier.  All
// wavefronts share one set of 64 rows per dot, cleared ahead of the kernel's main
// loop, and each sums whole columns, one row a lane; with 64 rows to clear, fill
// and sum for every wavefront (37 LDS operations a lane and dot instead of 12)
// this took about 4 us of kernel B at 128^3 (29.4 us; 25.1 without it).
template <int N, int K>
__device__ __forceinline__ void block_window(Dot<N> (&d)[K], const Shm<N>& s) {
  const int nw = blockDim.x >> 6, w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int j = 0; j < K; ++j) {
    double mx = 0.0;
#pragma unroll
    for (int k = 0; k < N; ++k) mx = fmax(mx, fabs(d[j].f.c[k]));
    const int top = wave_max_int((mx != 0.0) ? digits3_top(mx) : -1);
    if (lane == 0 && top >= 0) atomicMax(&s.imax[j], top);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const int top = s.imax[j];
    if (top >= 0)  // else the workgroup's sum of this dot is zero
      lane_deposit(d[j].f, top - (WIN - 1), s.scat + (j * 64 + lane) * ROW_STRIDE, s.sa + (size_t)j * SA_D, &s.flag[j]);
  }
  __syncthreads();
  if (__builtin_expect(nw < 4, 0)) {
    // few wavefronts for K WIN columns: a dot's columns at once, four lanes each (a
    // batch of 64 systems in tiles of 64 rows and workgroups of 64: 2.82 ms with one
    // column at a time, 2.50 so)
    const int col = lane % WIN, part = lane / WIN;
    for (int j = w; j < K; j += nw) {
      long long v = 0;
      if (lane < 4 * WIN)
        for (int r = part; r < 64; r += 4) v += s.scat[(j * 64 + r) * ROW_STRIDE + col];
      const long long a = __shfl(v, (lane + WIN) & 63, 64), b = __shfl(v, (lane + 2 * WIN) & 63, 64);
      v += a + b + __shfl(v, (lane + 3 * WIN) & 63, 64);
      if (lane < WIN) s.wsum[j * WIN + lane] = v;
    }
  } else {
    for (int c = w; c < K * WIN; c += nw) {
      const int j = c / WIN, k = c - j * WIN;
      const long long v = wave_sum_i64(s.scat[(j * 64 + lane) * ROW_STRIDE + k]);
      if (lane == 63) s.wsum[c] = v;
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Cross-workgroup reduction, finished by the last workgroup to arrive
// ---------------------------------------------------------------------------
// Every workgroup adds its part of each dot product into that dot's global long
// accumulator with device-scope integer atomics (its exact window digits, plus
// whatever went to its own long accumulator) and waits for their returned
// values, i.e. until they have been performed at the device's point of
// coherence.  Only then does it draw a ticket.  The workgroup that draws the last
// ticket reads and clears the accumulators with device-scope atomic exchanges,
// which observe every addition performed before, and rounds them.  No cache
// write-back fence is needed, and integer addition is associative, so the order
// of arrival cannot change the sum.  Plain FP64 mode: each workgroup publishes
// its block sum into its own slot the same way and the last one adds the G sums
// in workgroup order.
__device__ __forceinline__ unsigned long long dev_add(long long* p, long long v) {
  return __hip_atomic_fetch_add((unsigned long long*)p, (unsigned long long)v, __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
}

// Lightweight records: 8 components, tail, flags.
__device__ __forceinline__ void lw_pack(double (&v)[LW_REC], const Dot<LW8>& a) {
#pragma unroll
  for (int k = 0; k < LW_N; ++k) v[k] = a.f.c[k];
  v[LW_N] = a.tail;
  v[LW_N + 1] = (double)a.fl;
}

__device__ __forceinline__ void lw_store(double* r, const Dot<LW8>& a) {
  double v[LW_REC];
  lw_pack(v, a);
#pragma unroll
  for (int k = 0; k < LW_REC; ++k) r[k] = v[k];
}

// lanes that a merge of n records spans: a power of two
__device__ __forceinline__ int lw_width(int n) {
  int width = 1;
  while (width < n && width < 64) width <<= 1;
  return width;
}

// One wavefront merges the per-wave records (wave i at rec[(i*K + j)*LW_REC])
// of dot j; lane 0 ends with the workgroup's value.
__device__ __forceinline__ void lw_gather_waves(Dot<LW8>& a, const double* rec, int j, int K, int nw, int lane) {
  const bool in = lane < nw;
  const double* r = rec + (size_t)(lane * K + j) * LW_REC;
#pragma unroll
  for (int k = 0; k < LW_N; ++k) a.f.c[k] = in ? r[k] : 0.0;
  a.tail = in ? r[LW_N] : 0.0;
  a.fl = in ? (int)r[LW_N + 1] : 0;
  a.wave_merge(lw_width(nw));
}

// Every wavefront's record of each dot to LDS, then a barrier
template <int K>
__device__ __forceinline__ void lw_wave_records(Dot<LW8> (&d)[K], double* rec) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int j = 0; j < K; ++j) {
    d[j].wave_merge(64);
    if (lane == 0) lw_store(rec + (size_t)(w * K + j) * LW_REC, d[j]);
  }
  __syncthreads();
}

// Record b of dot j, published by another workgroup
__device__ __forceinline__ void lw_record(Dot<LW8>& a, const Red& red, int slot, int b) {
  const double* g = red.partials + ((size_t)slot * red.G + b) * LW_REC;
  double v[LW_REC];
#pragma unroll
  for (int k = 0; k < LW_REC; ++k)
    v[k] = __longlong_as_double(
        (long long)__hip_atomic_load((unsigned long long*)&g[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
#pragma unroll
  for (int k = 0; k < LW_N; ++k) a.f.c[k] = v[k];
  a.tail = v[LW_N];
  a.fl = (int)v[LW_N + 1];
}

// The rounded dot of a merged record (one thread)
__device__ __forceinline__ double lw_round(const Dot<LW8>& a) {
  double r = fpe_round(a.f);
  if (a.fl & F_LOST) r += a.tail;
  return (a.fl & F_NONFINITE) ? __longlong_as_double(0x7ff8000000000000ll) : r;
}

// Adds this workgroup's part of the K dots into the reduction slots slot0..
// (record b); returns a value that depends on every atomic's result.  Alone
// (without block_publish_last's ticket) it serves a reduction that the next
// kernel finishes: the end of this kernel then orders the atomics before it.
template <int N, int K>
__device__ __forceinline__ unsigned long long block_publish(Dot<N> (&d)[K], const Shm<N>& s, const Red& red,
                                                            int slot0, int b) {
  const int tid = threadIdx.x;
  unsigned long long sink = 0;
  if constexpr (N == LW8) {
    // twosum merge trees: lanes of each wave (shuffles), then the waves (LDS,
    // one wave per dot); lane 0 publishes the workgroup's record of each dot
    const int nw = blockDim.x >> 6, w = tid >> 6, lane = tid & 63;
    double* rec = (double*)s.wsum;
    lw_wave_records<K>(d, rec);
    for (int j = w; j < K; j += nw) {
      Dot<LW8> a;
      lw_gather_waves(a, rec, j, K, nw, lane);
      if (lane == 0) {
        double* g = red.partials + ((size_t)(slot0 + j) * red.G + b) * LW_REC;
        double v[LW_REC];
        lw_pack(v, a);
#pragma unroll
        for (int k = 0; k < LW_REC; ++k)
          sink += __hip_atomic_exchange((unsigned long long*)&g[k], (unsigned long long)__double_as_longlong(v[k]),
                                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  } else if constexpr (N > 0) {
    block_window<N, K>(d, s);
    long long* gsa = red.gsa + (size_t)(b & (red.copies - 1)) * (MAX_DOTS * SA_D);
    if (tid < K * WIN) {
      const int j = tid / WIN, k = tid % WIN;
      const int g = s.imax[j] - (WIN - 1) + k;
      const long long v = s.wsum[tid];
      if (s.imax[j] >= 0 && v != 0 && g >= 0 && g < SA_D) sink += dev_add(gsa + (size_t)(slot0 + j) * SA_D + g, v);
    }
    // rare: this workgroup's own long accumulators, and the non-finite flags
    if (tid < 64) {
      for (int j = 0; j < K; ++j) {
        const int fl = s.flag[j];
        if ((fl & F_NONFINITE) && tid == 0)
          sink += (unsigned)__hip_atomic_fetch_or(&red.gflags[slot0 + j], F_NONFINITE, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
        if (fl & F_SA) {
          long long* sa = s.sa + (size_t)j * SA_D;
          int lo, hi;
          sa_normalize_wave(sa, lo, hi);
          long long* g = gsa + (size_t)(slot0 + j) * SA_D;
          for (int k = lo + tid; k <= hi; k += 64)
            if (sa[k]) sink += dev_add(g + k, sa[k]);
        }
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const double v = plain_block_sum(d[j].s, s.pbuf);
      if (tid == 0)
        sink += __hip_atomic_exchange((unsigned long long*)&red.partials[(size_t)(slot0 + j) * red.G + b],
                                      (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  return sink;
}

// Returns true (in every thread) in the last workgroup to arrive.  `ticket`
// selects the arrival counter (kernels that run one after the other may share).
template <int N, int K>
__device__ __forceinline__ bool block_publish_last(Dot<N> (&d)[K], const Shm<N>& s, const Red& red, int slot0,
                                                   int b, int ticket) {
  const int tid = threadIdx.x;
  const unsigned long long sink = block_publish<N, K>(d, s, red, slot0, b);
  // using the returned values makes every thread wait until its atomics have
  // been performed before the barrier that precedes the ticket
  if (sink == 0x5bd1e9955bd1e995ull) s.misc[11] = 1;
  __syncthreads();
  if (tid == 0) {
    // true for the last of `of` workgroups to draw from *t, which it leaves zeroed
    auto draw = [](unsigned* t, unsigned of) {
      if (__hip_atomic_fetch_add(t, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != of - 1u) return false;
      __hip_atomic_exchange(t, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return true;
    };
    // the workgroups of each copy draw among themselves first, the last of each
    // copy then for the workgroup: 512 draws from one counter queue as 512
    // additions to one address do
    const unsigned c = (unsigned)(b & (red.copies - 1));
    const unsigned mine = ((unsigned)red.G - c + (unsigned)red.copies - 1u) / (unsigned)red.copies;
    bool last = true;
    if (red.copies > 1) last = draw(&red.tickets[kSubTickets + c], mine);
    if (last) last = draw(&red.tickets[ticket], red.copies > 1 ? (unsigned)red.copies : (unsigned)red.G);
    s.misc[10] = last;
  }
  __syncthreads();
  return s.misc[10] != 0;
}

// Exact dots: round the K long accumulators in s.sa (their flags in
// s.misc[1..K]) into s.res[0..K-1]; one wavefront per dot.  All threads call it.
template <int N, int K>
__device__ __forceinline__ void block_round_sa(const Shm<N>& s) {
  const int nw = blockDim.x >> 6, w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int j = w; j < K; j += nw) {  // one wave per dot
    const double r = sa_round(s.sa + (size_t)j * SA_D);
    if (lane == 0) s.res[j] = (s.misc[1 + j] & F_NONFINITE) ? __longlong_as_double(0x7ff8000000000000ll) : r;
  }
  __syncthreads();
}

// Item i of the K accumulators from slot0 on, all copies (0 <= i < K SA_D
// copies): its address, and the digit of s.sa it belongs to.
template <int K>
__device__ __forceinline__ unsigned long long* slot_item(const Red& red, int slot0, int i, int& digit) {
  const int c = i / (K * SA_D);
  digit = i - c * (K * SA_D);
  return (unsigned long long*)&red.gsa[(size_t)(c * MAX_DOTS + slot0) * SA_D + digit];
}

// How block_finalize reads the exact accumulators and flags.
enum : int {
  FIN_EXCHANGE = 0,  // the last workgroup to arrive: exchanges that leave them zeroed for the next use
  FIN_CLEAR = 1,     // a kernel after the one that published: loads, then stores of zero
  FIN_READ = 2       // the same, left for a later kernel to clear (block_clear_slots)
};

// Round the K dots of slots slot0.. into s.res[0..K-1] (their flags into
// s.misc[1..K]).
template <int N, int K, int Mode>
__device__ __forceinline__ void block_finalize(const Shm<N>& s, const Red& red, int slot0) {
  const int tid = threadIdx.x, bd = blockDim.x;
  if constexpr (N == LW8) {
    // A level of a merge is a chain of some 50 twosums (0.5 us), so records go
    // straight into lanes and only as many levels follow as there are records:
    // up to 64 of them in one wavefront a dot (n = 57 of a dot, one record: 13.3
    // us with all wavefronts merging all lanes, 8.0 in LDS; 1,000, two: 16.5, 11.7)
    const int nw = bd >> 6, w = tid >> 6, lane = tid & 63;
    if (red.G <= 64) {
      for (int j = w; j < K; j += nw) {
        Dot<LW8> a;
        a.zero();
        if (lane < red.G) lw_record(a, red, slot0 + j, lane);
        a.wave_merge(lw_width(red.G));
        if (lane == 0) {
          s.res[j] = lw_round(a);
          s.misc[1 + j] = a.fl;
        }
      }
      __syncthreads();
      return;
    }
    double* rec = (double*)s.wsum;
    const int held = min(nw, (red.G + 63) >> 6);  // wavefronts that hold records
    if (w < held) {
      for (int j = 0; j < K; ++j) {
        Dot<LW8> a;
        a.zero();
        if (tid < red.G) lw_record(a, red, slot0 + j, tid);
        for (int b0 = bd; b0 < red.G; b0 += bd) {  // all lanes absorb together
          Dot<LW8> c;
          c.zero();
          if (b0 + tid < red.G) lw_record(c, red, slot0 + j, b0 + tid);
          a.absorb(c.f.c, c.tail, c.fl);
        }
        a.wave_merge(64);
        if (lane == 0) lw_store(rec + (size_t)(w * K + j) * LW_REC, a);
      }
    }
    __syncthreads();
    for (int j = w; j < K; j += nw) {
      Dot<LW8> a;
      lw_gather_waves(a, rec, j, K, held, lane);
      if (lane == 0) {
        s.res[j] = lw_round(a);
        s.misc[1 + j] = a.fl;
      }
    }
    __syncthreads();
  } else if constexpr (N > 0) {
    for (int i = tid; i < K * SA_D; i += bd) s.sa[i] = 0;
    if (tid < K) {
      int* f = &red.gflags[slot0 + tid];
      if constexpr (Mode == FIN_EXCHANGE) {
        s.misc[1 + tid] = __hip_atomic_exchange(f, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        s.misc[1 + tid] = __hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (Mode == FIN_CLEAR) __hip_atomic_store(f, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    __syncthreads();
    constexpr int U = 4;  // items of a thread in flight
    for (int i0 = tid; i0 < K * SA_D * red.copies; i0 += U * bd) {
      unsigned long long v[U];
      int digit[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * bd;
        v[u] = 0ull;
        if (i < K * SA_D * red.copies) {
          unsigned long long* g = slot_item<K>(red, slot0, i, digit[u]);
          if constexpr (Mode == FIN_EXCHANGE)
            v[u] = __hip_atomic_exchange(g, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          else v[u] = __hip_atomic_load(g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (v[u] != 0ull) {
          lds_add(&s.sa[digit[u]], (long long)v[u]);
          if constexpr (Mode == FIN_CLEAR)
            __hip_atomic_store(slot_item<K>(red, slot0, i0 + u * bd, digit[u]), 0ull, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    block_round_sa<N, K>(s);
  } else {
    double v[K];
#pragma unroll
    for (int j = 0; j < K; ++j) v[j] = 0.0;
    for (int b = tid; b < red.G; b += bd)  // the loads of all K dots in flight together
#pragma unroll
      for (int j = 0; j < K; ++j)
        v[j] += __longlong_as_double((long long)__hip_atomic_load(
            (unsigned long long*)&red.partials[(size_t)(slot0 + j) * red.G + b], __ATOMIC_RELAXED,
            __HIP_MEMORY_SCOPE_AGENT));
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const double t = plain_block_sum(v[j], s.pbuf);
      if (tid == 0) s.res[j] = t;
    }
    __syncthreads();
  }
}

template <int N, int K>
__device__ __forceinline__ void block_finalize_last(const Shm<N>& s, const Red& red, int slot0) {
  block_finalize<N, K, FIN_EXCHANGE>(s, red, slot0);
}

// The only workgroup of a reduction (G = 1): round its K dots into
// s.res[0..K-1] (their flags into s.misc[1..K]) in LDS, with no accumulator in
// device memory.  The same bits as block_publish followed by
// block_finalize_last: an exact dot is the same integer (the window sums added
// to this workgroup's long accumulator instead of the global one) rounded
// once, a plain one the workgroup's sum plus zero, a lightweight one its record.
template <int N, int K>
__device__ __forceinline__ void block_reduce_local(Dot<N> (&d)[K], const Shm<N>& s) {
  const int tid = threadIdx.x;
  if constexpr (N == LW8) {
    const int nw = blockDim.x >> 6, w = tid >> 6, lane = tid & 63;
    lw_wave_records<K>(d, (double*)s.wsum);
    for (int j = w; j < K; j += nw) {
      Dot<LW8> a;
      lw_gather_waves(a, (const double*)s.wsum, j, K, nw, lane);
      if (lane == 0) {
        s.res[j] = lw_round(a);
        s.misc[1 + j] = a.fl;
      }
    }
    __syncthreads();
  } else if constexpr (N > 0) {
    block_window<N, K>(d, s);
    if (tid < K * WIN) {  // one (dot, digit) per thread: no two write one digit
      const int j = tid / WIN, k = tid % WIN;
      const int g = s.imax[j] - (WIN - 1) + k;
      const long long v = s.wsum[tid];
      if (s.imax[j] >= 0 && v != 0 && g >= 0 && g < SA_D) s.sa[(size_t)j * SA_D + g] += v;
    }
    if (tid < K) s.misc[1 + tid] = s.flag[tid] & F_NONFINITE;
    __syncthreads();
    block_round_sa<N, K>(s);
  } else {
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const double t = plain_block_sum(d[j].s, s.pbuf);
      if (tid == 0) s.res[j] = 0.0 + t;
    }
    __syncthreads();
  }
}

// Zero the exact accumulators and flags of slots slot0..slot0+K-1 (one
// workgroup; device-scope stores, so the atomics of a later kernel see them).
// Plain slots need nothing: every publication overwrites them.
template <int N, int K>
__device__ __forceinline__ void block_clear_slots(const Red& red, int slot0) {
  if constexpr (N > 0 && N != LW8) {
    for (int i = threadIdx.x; i < K * SA_D * red.copies; i += blockDim.x) {
      int digit;
      __hip_atomic_store(slot_item<K>(red, slot0, i, digit), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (threadIdx.x < K)
      __hip_atomic_store(&red.gflags[slot0 + threadIdx.x], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// A reduction published by the kernel before (exact dots), read by every
// workgroup of the next one: issue() starts the device-scope loads of the
// digits and flags into registers, so that the caller can start its own loads
// behind them; store() adds the copies up in s.sa and puts the flags in
// s.misc[1..K], ahead of a barrier and block_round_sa.
constexpr int DCAP = 5;  // items a thread loads ahead: all of two dots with 64 threads a copy
template <int N, int K>
struct Published {
  long long dg[DCAP];
  int fl;
  __device__ __forceinline__ void issue(const Shm<N>& s, const Red& red, int slot0) {
    const int items = K * SA_D * red.copies;
#pragma unroll
    for (int r = 0; r < DCAP; ++r) {
      const int i = threadIdx.x + r * blockDim.x;
      int digit;
      dg[r] = (i < items) ? (long long)__hip_atomic_load(slot_item<K>(red, slot0, i, digit), __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_AGENT)
                          : 0ll;
    }
    fl = (threadIdx.x < K) ? __hip_atomic_load(&red.gflags[slot0 + threadIdx.x], __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT)
                           : 0;
    for (int i = threadIdx.x; i < K * SA_D; i += blockDim.x) s.sa[i] = 0;
  }
  __device__ __forceinline__ void store(const Shm<N>& s, const Red& red, int slot0) const {
    const int items = K * SA_D * red.copies;
    __syncthreads();  // s.sa is cleared
#pragma unroll
    for (int r = 0; r < DCAP; ++r)
      if (dg[r] != 0) lds_add(&s.sa[(threadIdx.x + r * blockDim.x) % (K * SA_D)], dg[r]);
    for (int i = threadIdx.x + DCAP * blockDim.x; i < items; i += blockDim.x) {  // workgroups below 512 threads
      int digit;
      const long long v = (long long)__hip_atomic_load(slot_item<K>(red, slot0, i, digit), __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT);
      if (v != 0) lds_add(&s.sa[digit], v);
    }
    if (threadIdx.x < K) s.misc[1 + threadIdx.x] = fl;
  }
};

// ---------------------------------------------------------------------------
// Standalone exdot / plain dot and SpMV
// ---------------------------------------------------------------------------
template <int N>
__global__ void __launch_bounds__(1024) k_dot(long long n, const double* __restrict__ x,
                                              const double* __restrict__ y, double* out, int* lost, Red red) {
  extern __shared__ __align__(16) char smem[];
  Shm<N> s = shm_carve<N>(smem, 1, false);
  shm_init(s, 1);
  const int L = xcd_block(blockIdx.x, gridDim.x);
  long long chunk = (n + gridDim.x - 1) / gridDim.x;
  chunk = (chunk + 255) & ~255ll;
  long long lo = (long long)L * chunk, hi = lo + chunk;
  if (lo > n) lo = n;
  if (hi > n) hi = n;
  Dot<N> d[1];
  d[0].zero();
  // four elements at a time, all loads first: with one, a wavefront waited for
  // each pair of loads in turn (40M elements 143 us, 4.5 TB/s)
  constexpr int U = 4;
  long long i = lo + threadIdx.x;
  for (; i + (U - 1) * (long long)blockDim.x < hi; i += U * (long long)blockDim.x) {
    double a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      a[u] = x[i + u * (long long)blockDim.x];
      b[u] = y[i + u * (long long)blockDim.x];
    }
    if constexpr (N > 0 && N != LW8) {
      // what two insertions left over is added behind them, in one body: with one
      // behind every insertion 40M elements took 120 us, so 115
#pragma unroll
      for (int v = 0; v < U; v += 2) {
        const Left l = acc_insert(d[0].f, a[v], b[v]), r = acc_insert(d[0].f, a[v + 1], b[v + 1]);
        if (__builtin_expect(l.any() || r.any(), 0)) {
#pragma unroll 1
          for (int k = 0; k < 2; ++k) {
            const Left& w = k ? r : l;
            if (w.any()) acc_left<false>(w, a[v + k], b[v + k], s.sa, &s.flag[0]);
          }
        }
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) d[0].add(a[u], b[u], s.sa, &s.flag[0]);
    }
  }
  for (; i < hi; i += blockDim.x) d[0].add(x[i], y[i], s.sa, &s.flag[0]);
  if (gridDim.x == 1) {
    block_reduce_local<N, 1>(d, s);
  } else {
    if (!block_publish_last<N, 1>(d, s, red, 0, blockIdx.x, 0)) return;
    block_finalize_last<N, 1>(s, red, 0);
  }
  if (threadIdx.x == 0) {
    out[0] = s.res[0];
    if (lost) lost[0] = (N == LW8 && (s.misc[1] & F_LOST)) ? 1 : 0;
  }
}

template <int N, bool Win>
__global__ void __launch_bounds__(1024) k_spmv(Csr A, const double* __restrict__ x, double* __restrict__ y) {
  extern __shared__ __align__(16) char smem[];
  Shm<N> s = shm_carve<N>(smem, 0, true, Win ? A.win : 0);
  if constexpr (!Win) {
    pat_load(A, s);
    __syncthreads();
  }
  const int L = xcd_block(blockIdx.x, gridDim.x);
  const Range R = block_rows(A.n, L, gridDim.x);
  for_rows<N, Win>(A, GatherX{x}, R, s, [](int) { return 0; }, [&](int i, bool ok, double v, int) {
    if (ok) y[i] = v;
  });
}

}  // namespace rpk
