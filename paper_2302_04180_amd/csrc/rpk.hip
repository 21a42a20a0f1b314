// rpk.hip -- host side of the C ABI declared in include/rpk.h.
//
// Solver engine: the set-up kernels run once, then the iteration kernels are
// captured into a HIP graph holding a chunk of iterations.  Iterations run
// entirely on the device (scalars, stop test and status live in device memory);
// the host reads the 'done' flag once per chunk, and kernels of iterations past
// the stop are no-ops, so the result does not depend on the chunk size.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "host.h"
#include "setup.h"

using namespace rpk;
using namespace rpkhost;

// Reduction scratch of rpk_exdot_noalloc: one copy on every device the library
// runs on, held until the process ends.  Host code must not use this name as a
// device address: it is a host-side stand-in.  The address of each device's
// copy comes from hipGetSymbolAddress, taken once per device (noalloc_scratch).
// Holds the exdot workspace layout (header + per-workgroup partial records) of
// grids up to kScratchGrid workgroups.
constexpr size_t kScratchBytes = (size_t(1) << 20) + (size_t(1) << 16);
constexpr int kScratchGrid = 1624;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

struct Cfg {
  int block, grid, fpe, graph;
  int one;  // solve: every iteration in one workgroup (k_std_one / k_pcg_one)
};

rpk_status resolve(const rpk_launch* L, int64_t n, Cfg* c, bool scattered = false) {
  c->one = 0;
  const bool automatic = !L || (L->block == 0 && L->grid == 0);
  scattered = scattered && n >= kTinySolveRows;
  c->block = (L && L->block) ? L->block : (automatic && n >= (scattered ? kBigScatteredRows : kBigBlockRows)) ? 1024 : 512;
  c->fpe = (L && L->fpe) ? L->fpe : 3;
  c->graph = L ? L->graph : 0;
  if (c->block < 64 || c->block > 1024 || (c->block % 64) != 0) return RPK_ERR_ARG;
  if (c->fpe != 1 && c->fpe != 2 && c->fpe != 3 && c->fpe != 4 && c->fpe != 8) return RPK_ERR_ARG;
  if (c->graph < -1) return RPK_ERR_ARG;
  if (L && L->grid) {
    if (L->grid < 1 || L->grid > 65535) return RPK_ERR_ARG;
    c->grid = L->grid;
  } else {
    // 1,024 threads per CU of 256 CUs: few enough workgroups for their partial
    // sums to queue little, enough waves in flight for the streams (measured best
    // among 256..2048 workgroups of 256..1024 threads)
    int64_t need = (n + c->block - 1) / c->block;
    const int64_t most = automatic && (scattered || n >= kBigBlockRows) ? 256 : 512;
    if (automatic && scattered) need = most;
    if (need < 1) need = 1;
    if (need > most) need = most;
    if (need >= 8) need &= ~7ll;
    c->grid = (int)need;
  }
  // carry budget of the workgroups' long accumulators (a fixed small grid
  // cannot take a huge n)
  if ((n + c->grid - 1) / c->grid > kMaxPerGroup) return RPK_ERR_ARG;
  if (!records_fit(c->grid, c->block, c->fpe)) return RPK_ERR_ARG;
  return RPK_OK;
}

// Launch shape of a dot: that of the streaming kernels, but with the automatic
// shape one workgroup for short vectors, which reduces in LDS with no accumulator,
// ticket or second workgroup to wait for (not the lightweight ones), and for middle
// ones (kMidDot) fewer workgroups of two elements a thread.
rpk_status dot_shape(const rpk_launch* L, int64_t n, Cfg* c, bool light = false) {
  RET_IF(resolve(L, n, c));
  if (L && (L->block != 0 || L->grid != 0)) return RPK_OK;
  if (n <= (c->fpe > 1 ? kOneGroupDot : kOneGroupDotFpe1) && !light) {
    c->block = 1024;
    c->grid = 1;
  } else if (n >= kMidDot && n < kLongDot) {
    c->block = 512;
    c->grid = (int)std::min<int64_t>(kSmallSolveGroups, n / 1024 & ~7ll);
  }
  return RPK_OK;
}

// workspace header: state | tickets+flags | long accumulators | partials
struct Layout {
  size_t state, tickets, gflags, gsa, partials, vecs, total;
};

Layout layout(int grid, int64_t n, int nvec) {
  Layout l;
  size_t off = 0;
  l.state = off;
  off += up(sizeof(State));
  l.tickets = off;
  l.gflags = off + 8 * sizeof(unsigned);
  off += up(kTicketBytes);
  l.gsa = off;
  // room for every launch shape's copies: a workspace serves calls of different
  // shapes, and the partials of one must not lie on the accumulators of another
  off += up((size_t)kMaxCopies * MAX_DOTS * SA_D * sizeof(long long));
  l.partials = off;
  off += up((size_t)MAX_DOTS * grid * LW_REC * sizeof(double));  // plain sums / lightweight records per workgroup
  l.vecs = off;
  off += (size_t)nvec * up((size_t)n * sizeof(double));
  l.total = off;
  return l;
}

Red make_red(char* ws, const Layout& l, int grid) {
  Red r;
  r.partials = (double*)(ws + l.partials);
  r.gsa = (long long*)(ws + l.gsa);
  r.gflags = (int*)(ws + l.gflags);
  r.tickets = (unsigned*)(ws + l.tickets);
  r.G = grid;
  r.copies = red_copies(grid);
  return r;
}

template <int N>
struct DotF {
  static rpk_status call(int G, int B, hipStream_t s, long long n, const double* x, const double* y, double* o,
                         int* lost, Red r) {
    return Kern<N>::dot(G, B, s, n, x, y, o, lost, r);
  }
};
template <int N>
struct SpmvF {
  static rpk_status call(int G, int B, hipStream_t s, Csr A, const double* x, double* y) {
    return Kern<N>::spmv(G, B, s, A, x, y);
  }
};
template <int N>
struct InitF {
  static rpk_status call(int variant, int G, int B, hipStream_t s, Csr A, Vecs V, Red r) {
    return Kern<N>::init(variant, G, B, s, A, V, r);
  }
};
template <int N>
struct PhaseF {
  static rpk_status call(int variant, int ph, int G, int B, hipStream_t s, Csr A, Vecs V, Red r) {
    return Kern<N>::phase(variant, ph, G, B, s, A, V, r);
  }
};
// Iterations to launch before the next look at the state (automatic chunks).
// The residual's rate of decrease, since the last look and since the start,
// gives the iterations still needed (the smaller of the two estimates: Krylov
// convergence speeds up); the chunk is half of that plus one (a stop is taken
// by the first kernel of the iteration after it), so that the looks close in
// on the stop instead of overshooting it; twice the last chunk when there is no
// rate to go by; 1..kMaxChunk and not past maxit.  A surplus iteration costs
// launches that return at once (about 11 us on a small system), a look a host
// round trip (20-45 us); simulated on the residual histories of 7-point
// Poisson solves from 12^3 to 128^3 (standard and PCG) this costs about half of
// what the doubling chunks it replaced did.
int next_chunk(const State& h, int look_iter, double look_rel, int prev) {
  const double rel = h.tau / h.tau0;
  int c = 2 * prev;
  if (rel <= h.tol) {
    c = 1;
  } else if (h.iter > 0 && rel > 0.0 && rel < 1.0) {
    double need = std::log(h.tol / rel) / (std::log(rel) / h.iter);  // at the rate since the start
    if (h.iter > look_iter && rel < look_rel) {
      const double last = std::log(h.tol / rel) / (std::log(rel / look_rel) / (h.iter - look_iter));
      if (last < need) need = last;
    }
    if (need < 1e6) c = (int)std::ceil(0.5 * need) + 1;
  }
  if (c > kMaxChunk) c = kMaxChunk;
  if (c < 1) c = 1;
  const long long to_max = (long long)h.maxit - h.iter + 1;
  if (to_max >= 1 && c > to_max) c = (int)to_max;
  return c;
}

template <int N>
struct OneF {
  static rpk_status call(int variant, int B, hipStream_t s, Csr A, Vecs V, Red r, int iters) {
    return Kern<N>::one(variant, B, s, A, V, r, iters);
  }
};

// the instantiations of a single solve or dot: plain, exact (FPE length N) or lightweight
template <template <int> class F, typename... Args>
rpk_status by_dot(int N, Args&&... args) {
  if (N == LW8) return F<LW8>::call(args...);
  return by_fpe<F>(N, args...);
}

int kernel_n(int dots, int fpe) { return dots == RPK_DOT_PLAIN ? 0 : dots == RPK_DOT_FPE ? LW8 : fpe; }

// ---------------------------------------------------------------------------
// library-wide state
// ---------------------------------------------------------------------------
std::mutex g_mu;
std::map<std::vector<uint64_t>, hipGraphExec_t> g_graphs;
hipStream_t g_capture = nullptr;
State* g_pinned = nullptr;
size_t g_pinned_count = 0;

// Device address of this device's copy of `scratch` (rpk_exdot_noalloc), taken
// with hipGetSymbolAddress on the first call with that device current.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char* g_scratch[kMaxDevices] = {};

rpk_status noalloc_scratch(char** out) {
  int dev = -1;
  HIPCHK(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return RPK_ERR_HIP;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    HIPCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return RPK_ERR_HIP;
    g_scratch[dev] = (char*)p;
  }
  *out = g_scratch[dev];
  return RPK_OK;
}

}  // namespace

namespace rpkhost {

std::mutex& lib_mutex() { return g_mu; }
hipStream_t capture_stream() { return g_capture; }

rpk_status ensure_globals() {
  if (!g_capture) HIPCHK(hipStreamCreateWithFlags(&g_capture, hipStreamNonBlocking));
  if (!g_pinned) {
    HIPCHK(hipHostMalloc((void**)&g_pinned, sizeof(State), hipHostMallocDefault));
    g_pinned_count = 1;
  }
  return RPK_OK;
}

State* pinned_states(size_t count) {
  if (count > g_pinned_count) {
    State* p = nullptr;
    if (hipHostMalloc((void**)&p, count * sizeof(State), hipHostMallocDefault) != hipSuccess) return nullptr;
    if (g_pinned) (void)hipHostFree(g_pinned);
    g_pinned = p;
    g_pinned_count = count;
  }
  return g_pinned;
}

hipGraphExec_t graph_find(const std::vector<uint64_t>& key) {
  auto it = g_graphs.find(key);
  return it == g_graphs.end() ? nullptr : it->second;
}

void graph_put(const std::vector<uint64_t>& key, hipGraphExec_t g) {
  if (g_graphs.size() >= 256) {  // bound the cache: drop everything (rebuilt on demand)
    for (auto& kv : g_graphs) (void)hipGraphExecDestroy(kv.second);
    g_graphs.clear();
  }
  g_graphs[key] = g;
}

void graph_drop_owner(uint64_t owner) {
  for (auto it = g_graphs.begin(); it != g_graphs.end();) {
    if (!it->first.empty() && it->first[0] == owner) {
      (void)hipGraphExecDestroy(it->second);
      it = g_graphs.erase(it);
    } else {
      ++it;
    }
  }
}

}  // namespace rpkhost

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

const char* rpk_version(void) { return "rpk 0.1 (gfx950, exact FPE + long accumulator)"; }

const char* rpk_status_str(int32_t s) {
  switch (s) {
    case RPK_OK: return "RPK_OK";
    case RPK_ERR_ARG: return "RPK_ERR_ARG";
    case RPK_ERR_NOMEM: return "RPK_ERR_NOMEM";
    case RPK_ERR_HIP: return "RPK_ERR_HIP";
    case RPK_ERR_ZERO_DIAG: return "RPK_ERR_ZERO_DIAG";
    case RPK_ERR_NONFINITE: return "RPK_ERR_NONFINITE";
    case RPK_NOT_CONVERGED: return "RPK_NOT_CONVERGED";
    case RPK_BREAKDOWN: return "RPK_BREAKDOWN";
    case RPK_PENDING: return "RPK_PENDING";
    case RPK_REJECTED: return "RPK_REJECTED";
  }
  return "RPK_UNKNOWN";
}

static void free_matrix(rpk_matrix* A) {
  if (!A) return;
  if (A->rp) (void)hipFree(A->rp);
  if (A->ci) (void)hipFree(A->ci);
  if (A->v) (void)hipFree(A->v);
  if (A->dinv) (void)hipFree(A->dinv);
  if (A->sptr) (void)hipFree(A->sptr);
  if (A->scol) (void)hipFree(A->scol);
  if (A->sval) (void)hipFree(A->sval);
  if (A->sdif) (void)hipFree(A->sdif);
  if (A->dict) (void)hipFree(A->dict);
  delete A;
}

// Widest band (columns before and behind the row) of an operand window: 128 KB
constexpr int64_t kMaxBand = 16384;

// SELL-64 copy of the validated CSR (prefix sum of the slice widths, padded fill)
static rpk_status build_sell(rpk_matrix* A, const int* width, Band* band, hipStream_t s) {
  const int n = (int)A->n, ns = A->nslices;
  const size_t o_slim = (size_t)(ns + 1) * sizeof(long long), o_rlsb = o_slim + (size_t)ns * sizeof(int);
  if (hipMalloc((void**)&A->sptr, o_rlsb + (size_t)ns * 64) != hipSuccess) return RPK_ERR_NOMEM;
  A->slim = (int*)((char*)A->sptr + o_slim);
  A->rlsb = (signed char*)((char*)A->sptr + o_rlsb);
  long long total = 0;
  hipLaunchKernelGGL(k_slice_scan, dim3(1), dim3(1024), 0, s, width, ns, A->sptr);
  HIPCHK(hipGetLastError());
  HIPCHK(hipMemcpyAsync(&total, A->sptr + ns, sizeof(long long), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  A->sell_entries = total;
  const size_t cnt = (size_t)(total > 0 ? total : 1);
  if (hipMalloc((void**)&A->scol, cnt * sizeof(int)) != hipSuccess ||
      hipMalloc((void**)&A->sval, cnt * sizeof(double)) != hipSuccess)
    return RPK_ERR_NOMEM;
  const long long rows = (long long)ns * 64;
  hipLaunchKernelGGL(k_fill_sell, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, s, A->rp, A->ci, A->v, n, ns,
                     (const long long*)A->sptr, A->scol, A->sval, A->slim, A->rlsb);
  HIPCHK(hipGetLastError());
  // a tiny matrix is in the L1 caches: no window, and 25 of 215 us saved here
  if (A->n < kTinySolveRows) return RPK_OK;
  hipLaunchKernelGGL(k_band, dim3((unsigned)std::min(512, (ns + 3) / 4)), dim3(256), 0, s, n, ns,
                     (const long long*)A->sptr, (const int*)A->scol, band);
  HIPCHK(hipGetLastError());
  // operand window: where a gather touches at least 16 cache lines and a band of
  // columns leaves room for rows in LDS
  Band h;
  HIPCHK(hipMemcpyAsync(&h, band, sizeof(h), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  if (h.gathers == 0 || h.lines < 16 * (uint64_t)h.gathers || (int64_t)h.lo + h.hi > kMaxBand) return RPK_OK;
  if (hipMalloc((void**)&A->sdif, cnt * sizeof(unsigned short)) != hipSuccess) {
    (void)hipGetLastError();  // the matrix does without
    A->sdif = nullptr;
    return RPK_OK;
  }
  A->wlo = h.lo;
  A->whi = h.hi;
  hipLaunchKernelGGL(k_fill_dif, dim3((unsigned)std::min(4096, (ns + 3) / 4)), dim3(256), 0, s, n, ns,
                     (const long long*)A->sptr, (const int*)A->scol, h.lo, A->sdif);
  HIPCHK(hipGetLastError());
  return RPK_OK;
}

// Row dictionary (Csr::pid) where the matrix's rows are few different ones, as a
// stencil's are; the SELL copy is then not made.  The dictionary must fit the
// LDS set aside for it (kPatEntries) and a workgroup must read far fewer bytes
// for it than for its rows: at least 32 rows for each distinct one.  Byte
// offsets of a column and a slice's width must fit 32 bits and a byte.
// `found`, `pw`: the counters k_pat_find and k_slice_max left.
static rpk_status build_dictionary(rpk_matrix* A, int64_t found, int64_t pw, const int* width,
                                   const unsigned long long* hash, PatHash* t, hipStream_t s) {
  const int64_t np = found + 1;
  if (found > kPatMax || pw > 252 || np * pat_stride((int)pw) > kPatEntries || A->n < 32 * found || A->n > (1ll << 28))
    return RPK_OK;
  const size_t o_swid = up((size_t)A->nslices * 64), o_val = o_swid + up((size_t)A->nslices);
  if (hipMalloc((void**)&A->dict, o_val + (size_t)np * pat_stride((int)pw) * sizeof(PatEnt)) != hipSuccess)
    return RPK_ERR_NOMEM;
  A->pid = (unsigned char*)A->dict;
  A->swid = (unsigned char*)(A->dict + o_swid);
  A->pat = (PatEnt*)(A->dict + o_val);
  const unsigned G = (unsigned)std::min<int64_t>(2048, (A->nslices + 3) / 4);
  hipLaunchKernelGGL(k_pat_table, dim3(1), dim3(1024), 0, s, A->rp, A->ci, A->v, t, (int)np, (int)pw, A->pat);
  hipLaunchKernelGGL(k_pat_rows, dim3(G), dim3(256), 0, s, A->rp, A->ci, A->v, (int)A->n, A->nslices, width, hash, t,
                     (int)np, (int)pw, A->pat, A->pid, A->swid);
  HIPCHK(hipGetLastError());
  int fail = 0;
  HIPCHK(hipMemcpyAsync(&fail, &t->fail, sizeof(int), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  if (fail) {  // two different rows with one hash: the SELL copy serves them
    (void)hipFree(A->dict);
    A->dict = nullptr;
    A->pid = A->swid = nullptr;
    A->pat = nullptr;
  } else {
    A->np = (int)np;
    A->pw = (int)pw;
  }
  return RPK_OK;
}

// Scratch of a creation: what the host reads (Learned), the hash table's head behind it,
// slice widths; and n words that hold the rows' hashes, then the probe's x, in an
// allocation of their own.
// One copy tells the host what four did (262,144 different rows from device arrays 549 us
// before the row dictionary, 1,100 with four copies and one allocation just above 2 MiB, 425 so).
struct Learned {
  int flags[2];       // [0] row pointers, [1] entries
  unsigned probe[2];  // slices not certified, slices
  unsigned differ;    // the Jacobi vector is not uniform
  int pad;
  double d0;          // its first element
  Band band;
  int count, wide;    // head of the hash table
};
struct Setup {
  Learned* l;
  PatHash* t;  // at &l->count
  int* width;
  unsigned long long* words;
};

static rpk_status check_and_lay_out(rpk_matrix* A, const Setup& u, hipStream_t s) {
  const int n = (int)A->n, ns = A->nslices;
  const int B = 256;
  hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, s, (unsigned*)u.l, (long long)(offsetof(Learned, count) / sizeof(unsigned)));
  hipLaunchKernelGGL(k_pat_clear, dim3(1), dim3(1024), 0, s, u.t);
  hipLaunchKernelGGL(k_check_rowptr, dim3((unsigned)(((int64_t)n + 1 + B - 1) / B)), dim3(B), 0, s, A->rp, n,
                     (int)A->nnz, u.l->flags);
  HIPCHK(hipGetLastError());
  Learned h;
  HIPCHK(hipMemcpyAsync(&h, u.l, sizeof(int), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  if (h.flags[0]) return RPK_ERR_ARG;  // row_ptr unusable: do not read the rows
  const unsigned G = (unsigned)std::min(4096, (ns + 3) / 4);
  hipLaunchKernelGGL(k_setup_rows, dim3(G), dim3(256), 0, s, A->rp, A->ci, A->v, n, ns, A->dinv, u.width, u.words,
                     u.l->flags + 1);
  hipLaunchKernelGGL(k_slice_max, dim3(1), dim3(1024), 0, s, u.width, ns, &u.t->wide);
  hipLaunchKernelGGL(k_pat_find, dim3((unsigned)std::min<int64_t>(512, (A->n + 255) / 256)), dim3(256), 0, s, u.words,
                     n, u.t);
  // a uniform Jacobi vector (every dinv_i with the bits of dinv_0)
  hipLaunchKernelGGL(k_dinv_uniform, dim3((unsigned)(((int64_t)n + B - 1) / B)), dim3(B), 0, s, A->dinv, n,
                     &u.l->differ, &u.l->d0);
  HIPCHK(hipGetLastError());
  HIPCHK(hipMemcpyAsync(&h, u.l, sizeof(h), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  if (h.flags[1] & CHK_ARG) return RPK_ERR_ARG;
  if (h.flags[1] & CHK_NONFINITE) return RPK_ERR_NONFINITE;
  if (h.flags[1] & CHK_DIAG) return RPK_ERR_ZERO_DIAG;
  A->unif = h.differ == 0u ? 1 : 0;
  A->du = h.d0;
  RET_IF(build_dictionary(A, h.count, h.wide, u.width, u.words, u.t, s));
  if (!A->np) RET_IF(build_sell(A, u.width, &u.l->band, s));
  // Whether rows should try the certified row sum first: probe it on a
  // pseudo-random vector; not when more than one slice in eight has a row that it
  // cannot certify (results are the same either way).
  double* x = (double*)u.words;
  hipLaunchKernelGGL(k_fill_hash, dim3(1024), dim3(256), 0, s, x, (long long)n);
  hipLaunchKernelGGL(k_cert_probe, dim3(G), dim3(256), 0, s, csr_of(A), (const double*)x, u.l->probe);
  HIPCHK(hipGetLastError());
  HIPCHK(hipMemcpyAsync(h.probe, u.l->probe, sizeof(h.probe), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  A->cert = 8ull * h.probe[0] <= h.probe[1] ? 1 : 0;
  return RPK_OK;
}

static rpk_status create_impl(int64_t n, int64_t nnz, const int32_t* rp, const int32_t* ci, const double* v,
                              int32_t on_dev, hipStream_t s, rpk_matrix* A) {
  A->n = n;
  A->nnz = nnz;
  A->nslices = (int)((n + 63) / 64);
  if (hipMalloc((void**)&A->rp, (size_t)(n + 1) * 4) != hipSuccess) return RPK_ERR_NOMEM;
  if (hipMalloc((void**)&A->ci, (size_t)(nnz > 0 ? nnz : 1) * 4) != hipSuccess) return RPK_ERR_NOMEM;
  if (hipMalloc((void**)&A->v, (size_t)(nnz > 0 ? nnz : 1) * 8) != hipSuccess) return RPK_ERR_NOMEM;
  if (hipMalloc((void**)&A->dinv, (size_t)n * 8) != hipSuccess) return RPK_ERR_NOMEM;
  const hipMemcpyKind kind = on_dev ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
  HIPCHK(hipMemcpyAsync(A->rp, rp, (size_t)(n + 1) * 4, kind, s));
  if (nnz > 0) {
    HIPCHK(hipMemcpyAsync(A->ci, ci, (size_t)nnz * 4, kind, s));
    HIPCHK(hipMemcpyAsync(A->v, v, (size_t)nnz * 8, kind, s));
  }
  char* buf = nullptr;
  unsigned long long* words = nullptr;
  const size_t o_t = offsetof(Learned, count), o_width = up(o_t + sizeof(PatHash));
  static_assert(offsetof(Learned, wide) - offsetof(Learned, count) == offsetof(PatHash, wide) && offsetof(PatHash, count) == 0 &&
                offsetof(Learned, count) % alignof(PatHash) == 0, "Learned ends with the head of the hash table");
  if (hipMalloc((void**)&buf, o_width + (size_t)A->nslices * sizeof(int)) != hipSuccess) return RPK_ERR_NOMEM;
  rpk_status st = RPK_ERR_NOMEM;
  if (hipMalloc((void**)&words, (size_t)n * 8) == hipSuccess) {
    st = check_and_lay_out(A, Setup{(Learned*)buf, (PatHash*)(buf + o_t), (int*)(buf + o_width), words}, s);
    (void)hipFree(words);
  }
  (void)hipFree(buf);
  return st;
}

rpk_status rpk_matrix_create(int64_t n, int64_t nnz, const int32_t* row_ptr, const int32_t* col_idx,
                             const double* vals, int32_t ptrs_on_device, void* stream, rpk_matrix** out) {
  if (!out) return RPK_ERR_ARG;
  *out = nullptr;
  if (n < 1 || n >= (1ll << 31) || nnz < 0 || nnz >= (1ll << 31) || !row_ptr) return RPK_ERR_ARG;
  if (nnz > 0 && (!col_idx || !vals)) return RPK_ERR_ARG;
  rpk_matrix* A = new (std::nothrow) rpk_matrix();
  if (!A) return RPK_ERR_NOMEM;
  rpk_status st = create_impl(n, nnz, row_ptr, col_idx, vals, ptrs_on_device, (hipStream_t)stream, A);
  if (st != RPK_OK) {
    free_matrix(A);
    return st;
  }
  *out = A;
  return RPK_OK;
}

rpk_status rpk_matrix_destroy(rpk_matrix* A) {
  if (!A) return RPK_ERR_ARG;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    graph_drop_owner((uint64_t)(uintptr_t)A);
  }
  free_matrix(A);
  return RPK_OK;
}

rpk_status rpk_matrix_dims(const rpk_matrix* A, int64_t* n, int64_t* nnz) {
  if (!A) return RPK_ERR_ARG;
  if (n) *n = A->n;
  if (nnz) *nnz = A->nnz;
  return RPK_OK;
}

rpk_status rpk_matrix_dinv(const rpk_matrix* A, const double** dinv) {
  if (!A || !dinv) return RPK_ERR_ARG;
  *dinv = A->dinv;
  return RPK_OK;
}

rpk_status rpk_exdot_workspace_bytes(int64_t n, const rpk_launch* launch, size_t* bytes) {
  if (!bytes || n < 0) return RPK_ERR_ARG;
  Cfg c;
  RET_IF(resolve(launch, n, &c));
  *bytes = layout(c.grid, 0, 0).total;
  return RPK_OK;
}

rpk_status rpk_exdot(int64_t n, const double* x, const double* y, double* out_dev, int32_t dots,
                     const rpk_launch* launch_cfg, void* ws, size_t ws_bytes, void* stream) {
  if (n < 0 || n >= (1ll << 32) || !out_dev || !ws || (n > 0 && (!x || !y))) return RPK_ERR_ARG;
  if (dots != RPK_DOT_EXACT && dots != RPK_DOT_PLAIN) return RPK_ERR_ARG;
  Cfg c;
  RET_IF(dot_shape(launch_cfg, n, &c));
  const Layout l = layout(c.grid, 0, 0);
  if (ws_bytes < l.total) return RPK_ERR_ARG;
  Red red = make_red((char*)ws, l, c.grid);
  const int N = kernel_n(dots, c.fpe);
  return by_dot<DotF>(N, c.grid, c.block, (hipStream_t)stream, (long long)n, x, y, out_dev, (int*)nullptr, red);
}

rpk_status rpk_exdot_noalloc(int64_t n, const double* x, const double* y, double* out_dev, int32_t dots,
                             const rpk_launch* launch_cfg, void* stream) {
  if (n < 0 || n >= (1ll << 32) || !out_dev || (n > 0 && (!x || !y))) return RPK_ERR_ARG;
  if (dots != RPK_DOT_EXACT && dots != RPK_DOT_PLAIN) return RPK_ERR_ARG;
  Cfg c;
  RET_IF(dot_shape(launch_cfg, n, &c));
  const Layout l = layout(c.grid, 0, 0);
  if (c.grid > kScratchGrid || l.total > kScratchBytes) return RPK_ERR_ARG;  // beyond what the scratch array holds
  char* ws = nullptr;
  RET_IF(noalloc_scratch(&ws));
  hipStream_t s = (hipStream_t)stream;
  // tickets, flags and long accumulators start at zero (the kernel leaves them
  // zeroed; cleared all the same, by a kernel rather than a memset node); a
  // single workgroup uses none of them
  if (c.grid > 1) {
    hipLaunchKernelGGL(k_zero_words, dim3(32), dim3(256), 0, s, (unsigned*)ws,
                       (long long)(l.partials / sizeof(unsigned)));
    if (hipGetLastError() != hipSuccess) return RPK_ERR_HIP;
  }
  Red red = make_red(ws, l, c.grid);
  return by_dot<DotF>(kernel_n(dots, c.fpe), c.grid, c.block, s, (long long)n, x, y, out_dev, (int*)nullptr, red);
}

rpk_status rpk_fpedot(int64_t n, const double* x, const double* y, double* out_dev, int32_t* lost_dev,
                      const rpk_launch* launch_cfg, void* ws, size_t ws_bytes, void* stream) {
  if (n < 0 || n >= (1ll << 32) || !out_dev || !lost_dev || !ws || (n > 0 && (!x || !y))) return RPK_ERR_ARG;
  Cfg c;
  RET_IF(dot_shape(launch_cfg, n, &c, true));
  const Layout l = layout(c.grid, 0, 0);
  if (ws_bytes < l.total) return RPK_ERR_ARG;
  Red red = make_red((char*)ws, l, c.grid);
  return by_dot<DotF>(LW8, c.grid, c.block, (hipStream_t)stream, (long long)n, x, y, out_dev, (int*)lost_dev, red);
}

rpk_status rpk_exspmv(const rpk_matrix* A, const double* x, double* y, int32_t dots, const rpk_launch* launch_cfg,
                      void* stream) {
  if (!A || !x || !y || x == y) return RPK_ERR_ARG;
  if (dots != RPK_DOT_EXACT && dots != RPK_DOT_PLAIN && dots != RPK_DOT_FPE) return RPK_ERR_ARG;
  Cfg c;
  RET_IF(resolve(launch_cfg, A->n, &c, A->sdif != nullptr));
  const int N = (dots == RPK_DOT_PLAIN) ? 0 : c.fpe;  // the lightweight mode keeps the exact rows
  Csr Ac = csr_of(A);
  Ac.win = window_for(A, N, 0, c.grid, c.block);
  Ac.keep = keep_slices(A, 2, Ac.win != 0);  // repeated SpMVs of a matrix that fits reuse it from the cache
  return by_fpe<SpmvF>(N, c.grid, c.block, (hipStream_t)stream, Ac, x, y);
}

// Launch shape of a solve: that of the streaming kernels, except with the
// automatic shape (block and grid 0) on systems of fewer than kBigBlockRows rows: a
// standard or PCG solve with exact or plain dots of up to kOneGroupRows rows runs
// all its iterations in one workgroup of 1024 threads and one launch, and other
// solves, of matrices without scattered columns, take few large workgroups
// (kSmallSolveGroups).
static rpk_status solve_shape(const rpk_matrix* A, const rpk_opts* o, Cfg* c) {
  const bool automatic = o->launch.grid == 0 && o->launch.block == 0;
  rpk_launch L = o->launch;
  const bool scattered = A->sdif != nullptr && A->n >= kTinySolveRows;
  if (automatic && A->n < kBigBlockRows && !scattered) {
    const int64_t rows = A->n <= kShortSolveRows ? 128 : 256;
    const int64_t need = (A->n + rows - 1) / rows;
    L.block = A->n < kTinySolveRows ? 256 : 512;
    L.grid = (int32_t)std::min<int64_t>(kSmallSolveGroups, need < 8 ? need : (need + 7) & ~7ll);
  }
  if (automatic && A->n >= kBigBlockRows && !scattered && o->dots == RPK_DOT_PLAIN) {
    L.block = 512;  // see kBigBlockRows
    L.grid = 512;
  }
  RET_IF(resolve(&L, A->n, c, scattered));
  if (automatic && A->n <= kOneGroupRows && (o->variant == RPK_STD || o->variant == RPK_PCG) &&
      o->dots != RPK_DOT_FPE) {
    c->grid = 1;
    c->block = 1024;
    c->one = 1;
  }
  return RPK_OK;
}

rpk_status rpk_solve_workspace_bytes(const rpk_matrix* A, const rpk_opts* o, size_t* bytes) {
  if (!A || !o || !bytes) return RPK_ERR_ARG;
  if (o->variant != RPK_STD && o->variant != RPK_PIPELINED && o->variant != RPK_PCG) return RPK_ERR_ARG;
  Cfg c;
  RET_IF(solve_shape(A, o, &c));
  *bytes = layout(c.grid, A->n, nvec_of(o->variant)).total;
  return RPK_OK;
}

static Vecs carve_vecs(char* ws, const Layout& l, int64_t n, int variant, double* x, const double* b,
                       const rpk_opts* o) {
  Vecs V;
  std::memset(&V, 0, sizeof(V));
  const size_t step = up((size_t)n * sizeof(double));
  double* p[16];
  for (int k = 0; k < nvec_of(variant); ++k) p[k] = (double*)(ws + l.vecs + k * step);
  if (variant == RPK_PCG) {  // r, p, d (in s), y
    V.r = p[0]; V.p = p[1]; V.s = p[2]; V.y = p[3];
  } else {
    V.r0 = p[0]; V.r = p[1]; V.p = p[2]; V.ph = p[3]; V.s = p[4]; V.q = p[5]; V.qh = p[6]; V.y = p[7];
  }
  if (variant == RPK_PIPELINED) {
    V.rh = p[8]; V.w = p[9]; V.wh = p[10]; V.t = p[11]; V.sh = p[12]; V.z = p[13]; V.zh = p[14]; V.v = p[15];
  }
  V.x = x;
  V.b = b;
  V.st = (State*)(ws + l.state);
  V.hist = o->hist;
  V.xr = o->xr_hist;
  return V;
}

rpk_status rpk_solve(const rpk_matrix* A, const double* b, double* x, const rpk_opts* o, void* ws, size_t ws_bytes,
                     void* stream, rpk_info* info) {
  if (!A || !b || !x || !o || !ws || !info) return RPK_ERR_ARG;
  std::memset(info, 0, sizeof(*info));
  if (o->variant != RPK_STD && o->variant != RPK_PIPELINED && o->variant != RPK_PCG) return RPK_ERR_ARG;
  if (o->dots != RPK_DOT_EXACT && o->dots != RPK_DOT_PLAIN && o->dots != RPK_DOT_FPE) return RPK_ERR_ARG;
  if (o->maxit < 0 || !(o->tol >= 0.0)) return RPK_ERR_ARG;
  Cfg c;
  RET_IF(solve_shape(A, o, &c));
  const Layout l = layout(c.grid, A->n, nvec_of(o->variant));
  if (ws_bytes < l.total) return RPK_ERR_ARG;
  info->used.block = c.block;
  info->used.grid = c.grid;
  info->used.fpe = (o->dots == RPK_DOT_PLAIN) ? 0 : (o->dots == RPK_DOT_FPE) ? LW_N : c.fpe;
  info->used.graph = c.graph;
  const int loop = c.one ? LOOP5 : std_loop(A, o->variant, o->dots);
  info->streamed = streams_far(A, o->variant) ? 1 : 0;
  hipStream_t s = (hipStream_t)stream;
  std::lock_guard<std::mutex> lk(g_mu);
  RET_IF(ensure_globals());

  char* w = (char*)ws;
  const int variant = o->variant;
  const int N = kernel_n(o->dots, c.fpe);
  const int G = c.grid, B = c.block;
  const int nph = (variant == RPK_STD) ? 5 : (variant == RPK_PCG) ? 3 : 4;
  Red red = make_red(w, l, G);
  Vecs V = carve_vecs(w, l, A->n, variant, x, b, o);
  Csr Ac = csr_of(A);
  V.loop = loop;
  // the pipelined products have one more workgroup, which finishes the reduction before them
  if (!c.one)
    Ac.win = window_for(A, N, variant == RPK_STD ? 2 : variant == RPK_PCG ? 1 : 0,
                        std::max(1, G - (variant == RPK_PIPELINED ? 1 : 0)), B);
  V.far = info->streamed;
  V.near = rows_stay_near(A->n, variant, A->unif != 0) ? 1 : 0;
  Ac.keep = keep_slices(A, cached_vectors(variant, V.near != 0, V.far != 0, A->unif != 0), Ac.win != 0);

  const bool resume = o->resume != 0;
  // reduction scratch to zero; caller-visible histories to zero (not when resuming)
  if (!resume) hipLaunchKernelGGL(k_zero_words, dim3(16), dim3(256), 0, s, (unsigned*)(w + l.tickets),
                     (long long)((l.partials - l.tickets) / sizeof(unsigned)));
  HIPCHK(hipGetLastError());
  if (o->hist && !resume) {
    hipLaunchKernelGGL(k_fill, dim3(64), dim3(256), 0, s, o->hist, (long long)o->maxit * HIST_W, 0.0);
    HIPCHK(hipGetLastError());
  }
  if (o->xr_hist && !resume) {
    hipLaunchKernelGGL(k_fill, dim3(1024), dim3(256), 0, s, o->xr_hist, (long long)o->maxit * 2 * A->n, 0.0);
    HIPCHK(hipGetLastError());
  }
  if (variant == RPK_PIPELINED && !resume) {  // vectors of iteration -1 start at zero
    const size_t step = up((size_t)A->n * sizeof(double));
    hipLaunchKernelGGL(k_fill, dim3(1024), dim3(256), 0, s, (double*)(w + l.vecs),
                       (long long)(16 * step / sizeof(double)), 0.0);
    HIPCHK(hipGetLastError());
  }
  if (resume && loop == LOOP3) {
    hipLaunchKernelGGL(k_std_pair, dim3(256), dim3(256), 0, s, A->n, V, true);
    HIPCHK(hipGetLastError());
  }
  if (resume) hipLaunchKernelGGL(k_resume, dim3(1), dim3(64), 0, s, V.st, o->maxit);
  else hipLaunchKernelGGL(k_state_setup, dim3(1), dim3(64), 0, s, V.st, o->tol, o->maxit, variant);
  HIPCHK(hipGetLastError());

  hipEvent_t ev[RPK_NPHASE + 1] = {};
  const bool timing = o->timing != 0;
  if (timing)
    for (int k = 0; k <= RPK_NPHASE; ++k) HIPCHK(hipEventCreate(&ev[k]));
  auto cleanup = [&]() {
    if (timing)
      for (int k = 0; k <= RPK_NPHASE; ++k)
        if (ev[k]) (void)hipEventDestroy(ev[k]);
  };

  rpk_status st = RPK_OK;
  do {
    if (timing && hipEventRecord(ev[0], s) != hipSuccess) { st = RPK_ERR_HIP; break; }
    if (!resume) st = by_dot<InitF>(N, variant, G, B, s, Ac, V, red);
    if (st != RPK_OK) break;
    if (timing) {
      if (hipEventRecord(ev[1], s) != hipSuccess || hipEventSynchronize(ev[1]) != hipSuccess) { st = RPK_ERR_HIP; break; }
      float ms = 0.f;
      hipEventElapsedTime(&ms, ev[0], ev[1]);
      info->phase_ms[8] += ms;
      info->phase_launches[8] += 1;
    }
    if (hipMemcpyAsync(g_pinned, V.st, sizeof(State), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) { st = RPK_ERR_HIP; break; }
    const bool use_graph = !timing && c.graph >= 0;
    int chunk = c.graph > 0 ? c.graph : 4;
    int look_iter = g_pinned->iter;  // the state at the last look
    double look_rel = g_pinned->tau / g_pinned->tau0;
    long long launched = 0;
    while (!g_pinned->done) {
      // cannot happen: the device stops at maxit, in the first kernel of the
      // chunk after the one that ran the last iteration at the latest
      if (launched > (long long)o->maxit + 8) { st = RPK_ERR_HIP; break; }
      if (timing) {
        auto absent = [&](int ph) { return (loop == LOOP3 && ph == 0) || (loop != LOOP5 && ph == 2); };
        for (int ph = 0; ph < nph && st == RPK_OK; ++ph) {
          if (hipEventRecord(ev[ph], s) != hipSuccess) st = RPK_ERR_HIP;
          if (st == RPK_OK) st = by_dot<PhaseF>(N, variant, ph, G, B, s, Ac, V, red);
        }
        if (st != RPK_OK) break;
        if (hipEventRecord(ev[nph], s) != hipSuccess || hipEventSynchronize(ev[nph]) != hipSuccess) {
          st = RPK_ERR_HIP;
          break;
        }
        for (int ph = 0; ph < nph; ++ph) {
          if (absent(ph)) continue;
          float ms = 0.f;
          hipEventElapsedTime(&ms, ev[ph], ev[ph + 1]);
          info->phase_ms[ph] += ms;
          info->phase_launches[ph] += 1;
        }
        launched += 1;
      } else if (c.one) {
        // the kernel stops itself at the stop test, at maxit at the latest
        const int iters = o->maxit < INT_MAX ? o->maxit + 1 : INT_MAX;
        st = by_dot<OneF>(N, variant, B, s, Ac, V, red, iters);
        if (st != RPK_OK) break;
        launched += iters;
      } else if (use_graph) {
        // an automatic chunk as graphs of 64, 32, ..., 1 iterations (each
        // captured once), a fixed one as one graph
        for (int part = c.graph > 0 ? chunk : kMaxChunk; part >= 1 && st == RPK_OK; part >>= 1) {
          if (c.graph == 0 && !(chunk & part)) continue;
          const std::vector<uint64_t> key{(uint64_t)(uintptr_t)A, (uint64_t)(uintptr_t)b, (uint64_t)(uintptr_t)x,
                                          (uint64_t)(uintptr_t)ws, (uint64_t)(uintptr_t)o->hist,
                                          (uint64_t)(uintptr_t)o->xr_hist, (uint64_t)variant, (uint64_t)N,
                                          (uint64_t)G, (uint64_t)B, (uint64_t)part};
          hipGraphExec_t exec = nullptr;
          st = graph_get(key, [&](hipStream_t cs) {
            rpk_status cst = RPK_OK;
            for (int k = 0; k < part && cst == RPK_OK; ++k)
              for (int ph = 0; ph < nph && cst == RPK_OK; ++ph)
                cst = by_dot<PhaseF>(N, variant, ph, G, B, cs, Ac, V, red);
            return cst;
          }, &exec);
          if (st == RPK_OK && hipGraphLaunch(exec, s) != hipSuccess) st = RPK_ERR_HIP;
          if (c.graph > 0) break;
        }
        if (st != RPK_OK) break;
        launched += chunk;
      } else {
        const int k_iter = chunk;
        for (int k = 0; k < k_iter && st == RPK_OK; ++k)
          for (int ph = 0; ph < nph && st == RPK_OK; ++ph)
            st = by_dot<PhaseF>(N, variant, ph, G, B, s, Ac, V, red);
        if (st != RPK_OK) break;
        launched += k_iter;
      }
      if (hipMemcpyAsync(g_pinned, V.st, sizeof(State), hipMemcpyDeviceToHost, s) != hipSuccess ||
          hipStreamSynchronize(s) != hipSuccess) { st = RPK_ERR_HIP; break; }
      if (c.graph <= 0) {
        const int prev = chunk;
        chunk = next_chunk(*g_pinned, look_iter, look_rel, prev);
        look_iter = g_pinned->iter;
        look_rel = g_pinned->tau / g_pinned->tau0;
      }
    }
    if (st != RPK_OK) break;
    if (loop == LOOP3 && g_pinned->status == RPK_NOT_CONVERGED) {  // a checkpoint keeps p and s in place
      hipLaunchKernelGGL(k_std_pair, dim3(256), dim3(256), 0, s, A->n, V, false);
      if (hipGetLastError() != hipSuccess) { st = RPK_ERR_HIP; break; }
    }
    // reduction slots that a stop left published but not cleared (the kernels
    // that clear them did not run), so that the residual and a resumed solve
    // start from zeroed accumulators
    hipLaunchKernelGGL(k_zero_words, dim3(16), dim3(256), 0, s, (unsigned*)(w + l.tickets),
                       (long long)((l.partials - l.tickets) / sizeof(unsigned)));
    if (hipGetLastError() != hipSuccess) { st = RPK_ERR_HIP; break; }
    // true residual of the returned iterate, exact
    if (timing && hipEventRecord(ev[0], s) != hipSuccess) { st = RPK_ERR_HIP; break; }
    st = Kern<4>::resid(G, B, s, Ac, V, red);
    if (st != RPK_OK) break;
    if (timing) {
      if (hipEventRecord(ev[1], s) != hipSuccess || hipEventSynchronize(ev[1]) != hipSuccess) { st = RPK_ERR_HIP; break; }
      float ms = 0.f;
      hipEventElapsedTime(&ms, ev[0], ev[1]);
      info->phase_ms[9] += ms;
      info->phase_launches[9] += 1;
    }
    if (hipMemcpyAsync(g_pinned, V.st, sizeof(State), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) { st = RPK_ERR_HIP; break; }
  } while (0);
  cleanup();
  if (st != RPK_OK) return st;
  const State& h = *g_pinned;
  info->status = h.status;
  info->iters = h.iter;
  info->tau0 = h.tau0;
  info->tau = h.tau;
  info->true_res = h.true_res;
  info->inexact_dots = h.lost;
  return (rpk_status)h.status;
}

rpk_status rpk_matrix_form(const rpk_matrix* A, const rpk_launch* launch_cfg, int32_t form[4]) {
  if (!A || !form) return RPK_ERR_ARG;
  Cfg c;
  RET_IF(resolve(launch_cfg, A->n, &c, A->sdif != nullptr));
  const int loop = std_loop(A, RPK_STD, RPK_DOT_EXACT);
  form[0] = A->np ? A->np - 1 : 0;  // the last one is the empty row
  form[1] = window_for(A, c.fpe, 0, c.grid, c.block);
  form[2] = A->cert;
  form[3] = loop == LOOP3 ? 3 : loop == LOOP4 ? 4 : 5;
  return RPK_OK;
}

rpk_status rpk_device_divsqrt(int64_t n, const double* a, const double* b, double* q, double* r, void* stream) {
  if (n < 0 || (n > 0 && (!a || !b || !q || !r))) return RPK_ERR_ARG;
  if (n == 0) return RPK_OK;
  hipLaunchKernelGGL(k_divsqrt, dim3(1024), dim3(256), 0, (hipStream_t)stream, (long long)n, a, b, q, r);
  return hipGetLastError() == hipSuccess ? RPK_OK : RPK_ERR_HIP;
}

}  // extern "C"
