// setup.h -- non-template kernels used by the host code only (one translation unit).
#pragma once
#include "solver.h"

namespace rpk {

// ---------------------------------------------------------------------------
// Matrix set-up: checks and dinv_i = RN(1 / a_ii) (Sec. 4, Jacobi M = diag(A))
// ---------------------------------------------------------------------------
enum : int { CHK_ARG = 1, CHK_NONFINITE = 2, CHK_DIAG = 4 };

__global__ void k_check_rowptr(const int* rp, int n, int nnz, int* flags) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i > n) return;
  bool bad = false;
  if (i == 0 && rp[0] != 0) bad = true;
  if (i == n && rp[n] != nnz) bad = true;
  if (i < n && rp[i + 1] < rp[i]) bad = true;
  if (bad) atomicOr(flags, CHK_ARG);
}

// What a creation learns of the matrix: its distinct rows.
constexpr int kPatMax = 255;    // distinct rows (an id is a byte; the last id is the empty row)
constexpr int kPatSlots = 1024; // hash slots

// Limits of a row for the certified sum (CertLim), from its entries one after another.
struct RowLimits {
  int elo = INT_MAX, ehi = INT_MIN, lsb = INT_MAX;
  __device__ __forceinline__ void add(double v) {
    if (v == 0.0) return;
    bool neg;
    unsigned long long mant;
    int e;
    decode(v, neg, mant, e);
    const int top = e + 64 - __clzll((long long)mant);
    lsb = min(lsb, e + __ffsll((long long)mant) - 1);
    elo = min(elo, top);
    ehi = max(ehi, top);
  }
  __device__ __forceinline__ int pack() const { return elo == INT_MAX ? cert_pack(0, 0, 0) : cert_pack(elo, ehi, lsb); }
};

struct PatHash {
  int count;                          // distinct hashes so far (counts on past kPatMax)
  int wide;                           // widest slice
  int fail;                           // a row differs from its representative
  int pad;
  unsigned long long key[kPatSlots];  // 0 = free
  int rep[kPatSlots];                 // some row with that hash; k_pat_table: -1 - id
};

__device__ __forceinline__ unsigned long long pat_mix(unsigned long long v) {
  v *= 0x9E3779B97F4A7C15ull;
  v ^= v >> 29;
  v *= 0xBF58476D1CE4E5B9ull;
  return v ^ (v >> 32);
}

// The 64 rows of one slice as its wavefront sees them: their row pointers in
// LDS, and the row (0..63) that entry e of the CSR belongs to.
struct SliceRows {
  int rp[65];
  __device__ __forceinline__ void load(const int* g, int n, int s) {
    const int lane = threadIdx.x & 63;
    const int r = 64 * s + lane;
    rp[lane] = g[r < n ? r : n];
    if (lane == 0) rp[64] = g[slice_end(n, s)];
  }
  __device__ __forceinline__ int row_of(int e) const {
    int lo = 0;  // the last row that starts at or before e
#pragma unroll
    for (int step = 32; step >= 1; step >>= 1)
      if (rp[lo + step] <= e) lo += step;
    return lo;
  }
};

// One wavefront per slice, its lanes over the slice's entries (the loads
// coalesce whatever the rows' lengths; one row a thread took 3.1 ms on the
// 27-point 159^3 matrix): the checks of every entry, dinv, the slice's width
// and, for the row dictionary, each row's hash over its (position, column - row,
// value).  n entries of hash.
__global__ void __launch_bounds__(256) k_setup_rows(const int* rp, const int* ci, const double* v, int n, int nslices,
                                                    double* dinv, int* width, unsigned long long* hash, int* flags) {
  __shared__ SliceRows R[4];
  __shared__ unsigned long long h[4][64];
  __shared__ double diag[4][64];
  __shared__ int cnt[4][64];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int fl = 0;
  for (int s = blockIdx.x * 4 + w; s < nslices; s += gridDim.x * 4) {
    R[w].load(rp, n, s);
    h[w][lane] = 0ull;
    cnt[w][lane] = 0;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
    for (LaneEntries it(R[w].rp[0], R[w].rp[64], lane); it.more(); it.next()) {
      const int e = it.at(), l = R[w].row_of(e), r = 64 * s + l;
      const int c = ci[e];
      const double val = v[e];
      if (c < 0 || c >= n) fl |= CHK_ARG;
      if (!isfinite(val)) fl |= CHK_NONFINITE;
      if (c == r) {
        atomicAdd(&cnt[w][l], 1);
        diag[w][l] = val;
      }
      const unsigned long long at = ((unsigned long long)(unsigned)(e - R[w].rp[l]) << 32) | (unsigned)(c - r);
      atomicAdd(&h[w][l], pat_mix(pat_mix(at) ^ (unsigned long long)__double_as_longlong(val)));
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
    const int r = 64 * s + lane, len = R[w].rp[lane + 1] - R[w].rp[lane];
    if (r < n) {
      const bool one = cnt[w][lane] == 1 && diag[w][lane] != 0.0;
      if (!one) fl |= CHK_DIAG;
      dinv[r] = one ? 1.0 / diag[w][lane] : 0.0;
      hash[r] = pat_mix(h[w][lane] ^ (unsigned)len) | 1ull;  // 0 marks a free slot
    }
    const int wide = wave_max_int(r < n ? len : 0);
    if (lane == 0) width[s] = wide;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
  }
  if (fl) atomicOr(flags, fl);
}

// *differ = 1 when some dinv_i does not have the bits of dinv_0 (Csr::unif), *first = dinv_0
__global__ void k_dinv_uniform(const double* dinv, int n, unsigned* differ, double* first) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *first = dinv[0];
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const bool d = i < n && __double_as_longlong(dinv[i]) != __double_as_longlong(dinv[0]);
  // one store for the first workgroups that find a difference, not one of every lane
  if (__syncthreads_or(d) && threadIdx.x == 0 &&
      __hip_atomic_load(differ, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u)
    atomicOr(differ, 1u);
}

// Largest of the slices' widths (one workgroup of 1024).
__global__ void __launch_bounds__(1024) k_slice_max(const int* width, int nslices, int* out) {
  __shared__ int wmax;
  if (threadIdx.x == 0) wmax = 0;
  __syncthreads();
  int mine = 0;
  for (int i = threadIdx.x; i < nslices; i += 1024) mine = width[i] > mine ? width[i] : mine;
  atomicMax(&wmax, mine);
  __syncthreads();
  if (threadIdx.x == 0) *out = wmax;
}

// SELL-64 construction (see Csr): exclusive prefix sum of 64*width into
// sptr[0..nslices] (one workgroup of 1024) ...
__global__ void __launch_bounds__(1024) k_slice_scan(const int* width, int nslices, long long* sptr) {
  __shared__ long long buf[1024];
  long long carry = 0;
  for (int base = 0; base < nslices; base += 1024) {
    const int i = base + threadIdx.x;
    buf[threadIdx.x] = (i < nslices) ? 64ll * width[i] : 0ll;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
      const long long v = (threadIdx.x >= (unsigned)d) ? buf[threadIdx.x - d] : 0ll;
      __syncthreads();
      buf[threadIdx.x] += v;
      __syncthreads();
    }
    if (i < nslices) sptr[i + 1] = carry + buf[threadIdx.x];
    carry += buf[1023];
    __syncthreads();
  }
  if (threadIdx.x == 0) sptr[0] = 0;
}

// ... and the entries, padded with (0, own row); rows past n point at column 0.  The
// limits of each slice and row (CertLim).
__global__ void k_fill_sell(const int* rp, const int* ci, const double* v, int n, int nslices, const long long* sptr,
                            int* scol, double* sval, int* slim, signed char* rlsb) {
  const long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= (long long)nslices * 64) return;
  const int s = (int)(r >> 6), lane = (int)(r & 63);
  const long long off = sptr[s];
  const int w = (int)((sptr[s + 1] - off) >> 6);
  const int k0 = (r < n) ? rp[r] : 0, len = (r < n) ? rp[r + 1] - rp[r] : 0;
  RowLimits lim;
  for (int j = 0; j < w; ++j) {
    const long long at = off + 64ll * j + lane;
    if (j < len) {
      const double a = v[k0 + j];
      scol[at] = ci[k0 + j];
      sval[at] = a;
      lim.add(a);
    } else {
      scol[at] = (r < n) ? (int)r : 0;
      sval[at] = 0.0;
    }
  }
  rlsb[r] = cert_pack_lsb(lim.lsb == INT_MAX ? 0 : lim.lsb);
  const int elo = -wave_max_int(-lim.elo), ehi = wave_max_int(lim.ehi);  // the wavefront holds the slice
  if (lane == 0) slim[s] = cert_pack(elo, ehi, 0);
}

// For the operand window (Csr::win): how far columns lie before and behind their
// rows; the gathers of the SELL copy, and the lanes of them that leave the cache
// line of the lane before (or are the first).
struct Band {
  int lo, hi;
  unsigned lines, gathers;  // of every sixteenth slice
};
__global__ void __launch_bounds__(256) k_band(int n, int nslices, const long long* sptr, const int* scol, Band* band) {
  __shared__ Band sum;
  if (threadIdx.x == 0) sum = Band{0, 0, 0u, 0u};
  __syncthreads();
  const int lane = threadIdx.x & 63;
  int lo = 0, hi = 0;
  unsigned lines = 0, gathers = 0;
  for (int s = (blockIdx.x * blockDim.x + threadIdx.x) >> 6; s < nslices; s += gridDim.x * blockDim.x >> 6) {
    const int r = 64 * s + lane;
    for (long long at = sptr[s] + lane; at < sptr[s + 1]; at += 64) {
      const int c = r < n ? scol[at] : r;
      lo = max(lo, r - c);
      hi = max(hi, c - r);
      if ((s & 15) == 0) {
        const int before = __shfl_up(c, 1);
        lines += __popcll(__ballot(lane == 0 || (c >> 4) != (before >> 4)));
        ++gathers;
      }
    }
  }
  atomicMax(&sum.lo, lo);
  atomicMax(&sum.hi, hi);
  if (lane == 0) {
    atomicAdd(&sum.lines, lines);
    atomicAdd(&sum.gathers, gathers);
  }
  __syncthreads();
  if (threadIdx.x == 0) {  // one of each a workgroup
    atomicMax(&band->lo, sum.lo);
    atomicMax(&band->hi, sum.hi);
    atomicAdd(&band->lines, sum.lines);
    atomicAdd(&band->gathers, sum.gathers);
  }
}

// 16-bit distances of the entries for the operand window (padding: the own row)
__global__ void k_fill_dif(int n, int nslices, const long long* sptr, const int* scol, int wlo, unsigned short* sdif) {
  const int lane = threadIdx.x & 63;
  for (int s = (blockIdx.x * blockDim.x + threadIdx.x) >> 6; s < nslices; s += gridDim.x * blockDim.x >> 6) {
    const int r = 64 * s + lane;
    for (long long at = sptr[s] + lane; at < sptr[s + 1]; at += 64)
      sdif[at] = (unsigned short)(r < n ? scol[at] - r + wlo : wlo);
  }
}

// Row dictionary (Csr::pid).  A row is its list of (column - row, value) in CSR
// order; every distinct one is found by the 64-bit hash k_setup_rows took, in an
// open-addressing table, some row with a hash represents it, and every
// row is then compared with its representative entry by entry, so a hash
// collision only costs the dictionary, never a value.
__global__ void __launch_bounds__(1024) k_pat_clear(PatHash* t) {
  for (int i = threadIdx.x; i < kPatSlots; i += blockDim.x) {
    t->key[i] = 0ull;
    t->rep[i] = 0x7fffffff;
  }
  if (threadIdx.x == 0) {
    t->count = t->wide = t->fail = 0;
  }
}

// Enter every row's hash and note a row that has it.  Each workgroup
// takes a contiguous chunk of rows; a hash goes to the device's table once per
// wavefront that meets it first (its lowest lane) and then never again from
// that workgroup, which keeps the hashes it has entered in LDS: with every
// thread looking for itself, the hot words took 2.6 ms at 128^3.  Wavefronts
// stop once more than kPatMax different rows have been seen (a matrix without
// structure ends here after a few thousand rows).
__global__ void __launch_bounds__(256) k_pat_find(const unsigned long long* hash, int n, PatHash* t) {
  __shared__ unsigned long long seen[512];
  for (int i = threadIdx.x; i < 512; i += blockDim.x) seen[i] = 0ull;
  __syncthreads();
  const long long chunk = ((long long)n + gridDim.x - 1) / gridDim.x;
  const long long lo = blockIdx.x * chunk, hi = lo + chunk < n ? lo + chunk : n;
  for (long long r = lo + threadIdx.x; r < hi; r += blockDim.x) {
    const unsigned long long h = hash[r];
    unsigned long long todo = __ballot(seen[(h >> 8) & 511] != h);
    while (todo) {  // one lane for each different hash that is new here
      const int l = __ffsll((long long)todo) - 1;
      const unsigned long long hl = __shfl(h, l, 64);
      todo &= ~__ballot(h == hl);
      bool many = false;
      if ((int)(threadIdx.x & 63) == l) {
        int i = (int)(h >> 32) & (kPatSlots - 1);
        for (;; i = (i + 1) & (kPatSlots - 1)) {
          many = __hip_atomic_load(&t->count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > kPatMax;
          if (many) break;  // also when the table is full
          unsigned long long k = __hip_atomic_load(&t->key[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (k == 0ull) {
            k = atomicCAS(&t->key[i], 0ull, h);
            if (k == 0ull) atomicAdd(&t->count, 1);
          }
          if (k == 0ull || k == h) break;
        }
        if (!many) atomicMin(&t->rep[i], (int)r);
        seen[(h >> 8) & 511] = h;
      }
      if (__ballot(many)) return;
    }
  }
}

// One workgroup: number the distinct rows by the rows that represent them (which may
// differ from one creation to the next, and the numbers with them), and write the
// dictionary, its rows padded with (0, own element); id np - 1 is the empty row.
__global__ void __launch_bounds__(1024) k_pat_table(const int* rp, const int* ci, const double* v, PatHash* t, int np,
                                                    int pw, PatEnt* pat) {
  __shared__ int rep[kPatMax + 1];
  __shared__ int byid[kPatMax + 1];
  __shared__ int cnt;
  if (threadIdx.x == 0) cnt = 0;
  __syncthreads();
  for (int i = threadIdx.x; i < kPatSlots; i += blockDim.x)
    if (t->key[i]) rep[atomicAdd(&cnt, 1)] = t->rep[i];  // np - 1 <= kPatMax of them
  __syncthreads();
  for (int i = threadIdx.x; i < kPatSlots; i += blockDim.x)
    if (t->key[i]) {
      const int r = t->rep[i];
      int id = 0;
      for (int k = 0; k < cnt; ++k) id += rep[k] < r;
      byid[id] = r;
      t->rep[i] = -1 - id;
    }
  __syncthreads();
  const int stride = pat_stride(pw);
  for (int k = threadIdx.x; k < np * stride; k += blockDim.x) {
    const int id = k / stride, j = k - id * stride;
    const int r = id < np - 1 ? byid[id] : 0;
    const int k0 = rp[r], len = id < np - 1 ? rp[r + 1] - k0 : 0;
    int lim = 0;
    if (j == 0) {
      RowLimits l;
      for (int e = 0; e < len; ++e) l.add(v[k0 + e]);
      lim = l.pack();
    }
    pat[k] = j < len ? PatEnt{v[k0 + j], 8 * (ci[k0 + j] - r), lim} : PatEnt{0.0, 0, lim};
  }
}

// One wavefront per slice: every row's id and a comparison of its entries with
// that dictionary row, bit by bit; the slice's width.
__global__ void __launch_bounds__(256) k_pat_rows(const int* rp, const int* ci, const double* v, int n, int nslices,
                                                  const int* width, const unsigned long long* hash, PatHash* t, int np,
                                                  int pw, const PatEnt* pat, unsigned char* pid, unsigned char* swid) {
  __shared__ SliceRows R[4];
  __shared__ int id[4][64];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int stride = pat_stride(pw);
  bool bad = false;
  unsigned long long last = 0ull;
  int last_id = 0;
  for (int s = blockIdx.x * 4 + w; s < nslices; s += gridDim.x * 4) {
    R[w].load(rp, n, s);
    const int r = 64 * s + lane;
    int mine = np - 1;
    if (r < n) {
      const unsigned long long hr = hash[r];
      if (hr != last) {
        int i = (int)(hr >> 32) & (kPatSlots - 1);
        for (int probe = 0; probe < kPatSlots && t->key[i] != hr; ++probe) i = (i + 1) & (kPatSlots - 1);
        last = hr;
        last_id = t->key[i] == hr ? -1 - t->rep[i] : -1;
      }
      mine = last_id;
      if (mine < 0 || mine >= np - 1) {
        bad = true;
        mine = np - 1;
      } else {  // as long as the representative: it has an entry here and the padding behind it
        const int len = rp[r + 1] - rp[r];
        if (len > pw) {
          bad = true;
        } else {
          const PatEnt behind = pat[mine * stride + len];
          bad |= behind.a != 0.0 || behind.off8 != 0;
        }
      }
    }
    id[w][lane] = mine;
    pid[(size_t)64 * s + lane] = (unsigned char)mine;
    if (lane == 0) swid[s] = (unsigned char)width[s];
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
    for (LaneEntries it(R[w].rp[0], R[w].rp[64], lane); it.more(); it.next()) {
      const int e = it.at(), l = R[w].row_of(e);
      const int j = e - R[w].rp[l];
      const PatEnt p = pat[id[w][l] * stride + (j < pw ? j : 0)];
      bad |= j >= pw || 8 * (ci[e] - (64 * s + l)) != p.off8 ||
             __double_as_longlong(v[e]) != __double_as_longlong(p.a);
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
  }
  if (__ballot(bad) && lane == 0) atomicOr(&t->fail, 1);
}

// Probe at matrix creation: counts[0] += slices where row_cert did not certify
// some row on x, counts[1] += slices.  Workgroups count in LDS first: an atomic
// of every wavefront on the same words took most of the probe's time (128^3:
// 755 us).
__global__ void __launch_bounds__(256) k_cert_probe(Csr A, const double* __restrict__ x, unsigned* counts) {
  __shared__ unsigned mine[2];
  if (threadIdx.x < 2) mine[threadIdx.x] = 0u;
  __syncthreads();
  const int nslices = (A.n + 63) >> 6;
  const int lane = threadIdx.x & 63;
  for (int s = (int)((blockIdx.x * (size_t)blockDim.x + threadIdx.x) >> 6); s < nslices;
       s += (int)((gridDim.x * (size_t)blockDim.x) >> 6)) {  // whole wavefronts
    double y;
    const int row = (s << 6) + lane;
    bool c;
    if (A.np) {  // the dictionary read from device memory
      const PatSrc src{A.pat, (unsigned)(row < A.n ? row : A.n - 1) * 8u, (int)A.pid[row] * pat_stride(A.pw)};
      c = row_cert(PatLim{A.pat + src.at0}, src, GatherX{x}, A.swid[s], y);
    } else {
      const long long off = A.sptr[s];
      const SellSrc<true> src{A.sval + off, A.scol + off};
      c = row_cert(SellLim(A, s, row), src, GatherX{x}, (int)((A.sptr[s + 1] - off) >> 6), y);
    }
    const bool fail = __ballot(row < A.n && !c) != 0ull;
    if (lane == 0) {
      atomicAdd(&mine[1], 1u);
      if (fail) atomicAdd(&mine[0], 1u);
    }
  }
  __syncthreads();
  if (threadIdx.x < 2 && mine[threadIdx.x]) atomicAdd(&counts[threadIdx.x], mine[threadIdx.x]);
}

// x[i] in [-1, 1) from a 64-bit mix of i (the certified-row probe's input)
__global__ void k_fill_hash(double* x, long long n) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    unsigned long long z = (unsigned long long)i * 0x9E3779B97F4A7C15ull + 0x632BE59BD9B4E019ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    x[i] = (double)(z >> 11) * 0x1p-52 - 1.0;
  }
}

__global__ void k_fill(double* p, long long n, double v) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    p[i] = v;
}

__global__ void k_zero_words(unsigned* p, long long n) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    p[i] = 0u;
}

// scalar IEEE division and square root as used by the solver's scalar steps
__global__ void k_divsqrt(long long n, const double* a, const double* b, double* q, double* r) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    q[i] = a[i] / b[i];
    r[i] = sqrt(a[i]);
  }
}

__global__ void k_state_setup(State* st, double tol, int maxit, int variant) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    State z = {};
    z.tol = tol;
    z.maxit = maxit;
    z.variant = variant;
    *st = z;
  }
}

// Between a checkpoint, where p and s are in place and p = r0 before the first
// iteration, as in the other loops, and the buffers of the three-kernel loop:
// enter before k_resume, leave at the iteration limit
__global__ void k_std_pair(int n, Vecs V, bool enter) {
  State* st = V.st;
  const int it = st->iter;
  const bool odd = (it & 1) != 0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    if (enter) {
      if (odd) {
        V.ph[i] = V.p[i];
        V.qh[i] = V.s[i];
      } else if (it == 0) {
        V.p[i] = 0.0;
        V.s[i] = 0.0;
      }
    } else if (odd) {
      V.p[i] = V.ph[i];
      V.s[i] = V.qh[i];
    } else if (it == 0) {
      V.p[i] = V.r[i];
    }
  }
  if (enter && blockIdx.x == 0 && threadIdx.x == 0) {
    st->iter_n = it;
    st->stg = st->rho;
  }
}

// Resume a solve stopped at its iteration limit (device state from the same
// workspace): continue up to `maxit` iterations in total.  A solve that stopped
// for any other reason keeps its status; one whose next step breaks down now
// reports the breakdown, as the uninterrupted solve would have.
__global__ void k_resume(State* st, int maxit) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  if (!st->done || st->status != ST_NOT_CONVERGED || maxit <= st->iter) return;
  if (st->resumable == 1) {
    st->done = 0;
    st->status = 0;
    st->maxit = maxit;
    st->resumable = 0;
  } else if (st->resumable == 2) {
    st->status = ST_BREAKDOWN;
    st->resumable = 0;
  }
}

}  // namespace rpk
