// host.h -- host-side pieces shared by the single-system solver (rpk.hip), the
// batched solver (batch.hip) and the request server (server.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <map>
#include <mutex>
#include <vector>

#include "kern.h"
#include "rpk.h"

struct rpk_matrix {
  int64_t n = 0, nnz = 0;
  int* rp = nullptr;  // CSR as given (validated), kept for reference
  int* ci = nullptr;
  double* v = nullptr;
  double* dinv = nullptr;
  int nslices = 0;    // SELL-64 copy used by the kernels
  long long* sptr = nullptr;
  int* scol = nullptr;
  double* sval = nullptr;
  long long sell_entries = 0;      // entries of the SELL copy, padding included
  unsigned short* sdif = nullptr;  // distances for the operand window (see Csr), absent where none pays
  int wlo = 0, whi = 0;
  char* dict = nullptr;            // row dictionary (see Csr), one allocation; sptr, scol and sval are then absent
  unsigned char* pid = nullptr;
  unsigned char* swid = nullptr;
  rpk::PatEnt* pat = nullptr;
  int np = 0, pw = 0;
  int cert = 0;                    // rows try the certified sum (see Csr)
  int* slim = nullptr;             // limits of slices and rows, behind sptr in its allocation
  signed char* rlsb = nullptr;
  int unif = 0;                    // every dinv_i has the bits of du (see Csr)
  double du = 0.0;
};

namespace rpkhost {

using namespace rpk;

#define HIPCHK(call)                              \
  do {                                            \
    if ((call) != hipSuccess) return RPK_ERR_HIP; \
  } while (0)

constexpr size_t kAlign = 256;
inline size_t up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Carry budget of the exact reductions.  Long-accumulator digits are int64
// words that receive signed 32-bit chunks and propagate no carry until the final
// rounding, so the number of chunks a digit can receive is what bounds a sum
// (Sec. 3.2 bounds the merges of its 52+12 split the same way):
//   - a workgroup's LDS accumulator takes, per digit, at most two chunks per
//     product it sums (the twoprod terms p and e) plus one per FPE component it
//     flushes: kMaxPerGroup elements per workgroup keep 2^30 + 8*1024 chunks of
//     < 2^32 below 2^63;
//   - a global accumulator takes, per digit and per published record, at most
//     one chunk per FPE component of every lane that had data, plus one digit of
//     the workgroup's normalised LDS accumulator: a reduction of R records from
//     L lanes with FPE length N stays below 2^63 when R (L N + 1) < 2^31.
// Single solves always fit the second rule (grid <= 65535, L <= 1024, N <= 8);
// the batched solver and the server check it per system (records = tiles).
constexpr int64_t kMaxPerGroup = int64_t(1) << 29;
// Solves of at most this many rows with the automatic launch shape run in one
// workgroup (standard and PCG loops, exact and plain dots): with exact dots
// measured faster at 512 rows and slower from 1,000 on, where one CU's share of
// the exact rows and dots outweighs the launches it saves (the pipelined loop
// ran slower in one workgroup already at 512 rows)
constexpr int64_t kOneGroupRows = 512;
// Solves of fewer than kBigBlockRows rows with the automatic launch shape take
// workgroups of 512 threads for 256 rows each (128 up to 4,096 rows), at most 248
// of them: the threads beyond the rows shorten the fixed parts of a kernel
// (clearing and reducing accumulators, the partial sums of the deferred points),
// one workgroup a CU has few partial sums to queue, and below 256 workgroups the
// accumulators have four copies to read instead of eight.  Fewer than 1,024 rows
// keep 256 threads, for 128 rows each.  40 iterations, pipelined / standard / PCG,
// us, in 256 threads for 256 rows (512 for 512 rows from 65,536 on, at most 512
// workgroups) and in this shape: 9^3 1,065 / 1,211 / 791 and 1,030 / 1,185 / 784,
// 16^3 1,121 / 1,091 / 789 and 1,005 / 1,036 / 764, 28^3 1,248 / 1,207 / 862 and
// 1,079 / 1,073 / 789, 56^3 1,598 / 1,482 / 982 and 1,400 / 1,287 / 911; 68^3 1,649 /
// 1,524 / 989 (256 of 1,024) and 1,752 / 1,499 / 991.
constexpr int64_t kTinySolveRows = 1024;
constexpr int64_t kShortSolveRows = 4096;
constexpr int64_t kSmallSolveGroups = 248;
// Dots of at most this many elements with the automatic launch shape run in one
// workgroup: 1,000 elements 4.3 us against 5.4 in two workgroups of 512.  With FPEs of
// one component nearly every term goes to the long accumulator, which one workgroup
// adds to at 3 us for 1,024 elements (a call of 4,096: 16.0 us, in eight workgroups 8.4).
constexpr int64_t kOneGroupDot = 4096, kOneGroupDotFpe1 = 1024;
// Dots of kMidDot to kLongDot - 1 elements with the automatic launch shape take
// workgroups of 512 threads for 1,024 elements each, at most kSmallSolveGroups: a
// call with up to 512 workgroups of 512 (256 of 1,024 from 262,144 elements on) and
// in this shape, exact / plain / lightweight, us: 128,000 elements 8.2 / 7.5 / 19.2
// and 7.7 / 7.3 / 17.9, 262,143 12.3 / 10.5 / 26.0 and 9.0 / 7.5 / 20.2, 500,000 10.1 /
// 8.0 / 24.2 and 9.7 / 7.7 / 21.4; exact at 1M 10.6 and 10.5, at 2M 12.4 and 12.8;
// below 65,536 the same within 2 %
constexpr int64_t kMidDot = 65536, kLongDot = 1 << 20;
// From this many rows on the automatic shape is 256 workgroups of 1,024 threads
// instead of 512 of 512 (solves: see kSmallSolveGroups; dots: kLongDot): as many
// wavefronts, but half the partial sums that queue on the accumulators (128^3 solve: B
// 25.0 and 23.5, D 30.6 and 28.0 us, 101^3 PCG: S1 15.8 and 14.6, S3 17.5 and 16.6 us).
// Solves with plain dots have no accumulators and keep 512 of 512: 24 iterations of
// 128^3 rows without a dictionary 3,573 us in 256 of 1,024, 3,481 so.
constexpr int64_t kBigBlockRows = 262144;
// Matrices of scattered columns (rpk_matrix::sdif) of at least kTinySolveRows rows
// take 256 workgroups, of 512 threads and from this many rows on of 1,024: their gathers keep a
// CU's L1 or LDS busy, so all CUs must share them, and one workgroup a CU leaves
// room for the operand window.  SpMV in the shape above and in this one, us:
// 30,000 rows (20 entries each) 8.6 and 5.5, 66,000 7.9 and 5.6, 130,000 10.2 and
// 7.5, 200,000 16.7 and 11.5 (with 512 threads 12.8)
constexpr int64_t kBigScatteredRows = 131073;
// Largest automatic chunk of iterations between two looks at a solve's state
constexpr int kMaxChunk = 64;
// Workgroups of one launch over a tile table (the rest take further launches):
// with 1,024 threads each, well inside a launch's 2^32 threads
constexpr int kMaxTileGrid = 1 << 20;
constexpr int64_t kCarryChunks = (int64_t(1) << 31) - 1;
inline bool records_fit(int64_t records, int64_t lanes, int fpe) {
  return records * (lanes * (int64_t)fpe + 1) <= kCarryChunks;
}

inline Csr csr_of(const rpk_matrix* A) {
  return Csr{A->sptr, A->scol, A->sval, A->dinv, (int)A->n, A->cert, A->slim, A->rlsb, 0, A->unif, A->du,
             A->pid, A->swid, A->pat, A->np, A->pw, A->sdif, A->wlo, A->whi, 0};
}

// Operand window (Csr::win) for G workgroups of B threads that share the rows in
// a kernel of K dots: where the matrix has distances, the window fits a CU's LDS
// with all workgroups resident at once, and each of its elements is gathered once
// on average.  20 scattered entries a row, SpMV, without and with it, us: 270,000
// rows 17.4 and 13.3, 500,000 27.0 and 19.6, 1,000,000 76.4 and 35.6; 200,000 rows
// in 512 workgroups, which would not all be resident, 16.7 and 20.0.
constexpr size_t kLdsBytes = 160 * 1024;
inline int window_for(const rpk_matrix* A, int N, int K, int G, int B) {
  if (!A->sdif) return 0;
  const int64_t chunk = (A->n + G - 1) / G;
  const int64_t win = ((chunk + 63) & ~63ll) + A->wlo + A->whi;
  if (win > (int64_t)(kLdsBytes / 8) || win * G > A->nnz) return 0;
  const size_t shm = shm_bytes(N, K, true, B, (int)win);
  if (shm > kLdsBytes || G > (int64_t)(256 * (kLdsBytes / shm))) return 0;
  return (int)win;
}

inline int nvec_of(int variant) { return variant == RPK_STD ? 8 : variant == RPK_PCG ? 4 : 16; }

// MI355X's Infinity Cache: 256 MiB in front of HBM, shared by all XCDs.
constexpr double kInfinityCacheBytes = 256.0 * 1024 * 1024;

// Leading SELL slices of A read with ordinary loads (Csr::keep): as much of
// the matrix as fits in nine tenths of the Infinity Cache next to `nvec`
// n-vectors (those one solver iteration touches, or x and y of a lone SpMV),
// so that the next SpMV finds it there.  Slices are counted in proportion to
// the SELL entries; none where a row dictionary replaces them.
inline int keep_slices(const rpk_matrix* A, int nvec, bool win) {
  if (A->np) return 0;
  const double vecs = (double)nvec * (double)A->n * 8.0;
  const double room = 0.9 * kInfinityCacheBytes - vecs;
  const double sell = (double)A->sell_entries * (win ? 10.0 : 12.0);
  if (room <= 0.0 || sell <= 0.0) return 0;
  if (room >= sell) return A->nslices;
  return (int)((double)A->nslices * (room / sell));
}

// Vectors one standard iteration touches: its eight work vectors, x and the
// Jacobi vector; with a uniform Jacobi vector p^ and q^ are never stored and
// dinv is a scalar, which leaves seven.  (The three-kernel loop has a second p and
// s; it runs where all fit.)
inline int std_vectors(bool unif) { return unif ? 7 : nvec_of(RPK_STD) + 2; }
// Loop of a single standard solve (Vecs::loop).  The shorter loops need a uniform
// Jacobi vector and a row dictionary, and the deferred reduction points.  They save
// a launch and a pass over vectors and pay with one (D3) or two (B3) more gathers
// per entry: about 0.37 us for a million entries in D3 against 4 us and 3.4 us for
// a million rows in C.  Measured, us: D3 and D + C 34.9 and 40.6 (128^3, 7 points),
// 17.2 and 19.2 (64^3, 27 points), 26.2 and 25.4 (80^3, 27), 76.4 and 68.4
// (128^3, 27); B3 and A + B, with 1 us for the gap between two kernels, 11.6 and
// 13.8 (64^3, 7), 16.8 and 17.4 (80^3, 7: 3.6M entries), 14.2 and 14.0 (48^3, 27:
// 3.0M), 43.4 and 39.2 (128^3, 7).
inline int std_loop(const rpk_matrix* A, int variant, int dots) {
  if (variant != RPK_STD || dots == RPK_DOT_FPE || A->unif == 0 || A->np == 0) return LOOP5;
  if (A->nnz <= 3000000) return LOOP3;
  return A->nnz <= 8000000 + 9 * (int64_t)A->n ? LOOP4 : LOOP5;
}
// Vectors the pipelined loop keeps cached when they fit: p^, q, q^, y, r, r^, w,
// t, v and z^, w^ (its other six, s, s^, z, x, r0 and dinv, are streamed unless
// all fit); with a uniform Jacobi vector z^ and w^ are never stored and z
// (gathered by P2) is kept instead: ten.
inline int pipe_kept(bool unif) { return unif ? 10 : 11; }

// Whether a solve streams vectors past the Infinity Cache, in the pipelined loop
// beyond the six (Vecs::far): the standard loop when the vectors it touches do not fit in
// nine tenths of the cache, the pipelined loop when the eleven it otherwise
// keeps do not.  A batch of systems decides the same way on its total number of
// rows (unif: every system's Jacobi vector is uniform).
inline bool rows_stream_far(int64_t rows, int variant, bool unif) {
  const int kept = variant == RPK_STD ? std_vectors(unif) : variant == RPK_PIPELINED ? pipe_kept(unif) : 0;
  return kept > 0 && (double)kept * (double)rows * 8.0 > 0.9 * kInfinityCacheBytes;
}
inline bool streams_far(const rpk_matrix* A, int variant) { return rows_stream_far(A->n, variant, A->unif != 0); }
// Whether the pipelined loop streams nothing (Vecs::near): all the vectors it
// touches, seventeen, or fourteen with a uniform Jacobi vector, fit in nine tenths
// of the cache.  P1 and P3 without and with the six always-streamed ones kept, us:
// 96^3 28.3 + 21.4 and 25.2 + 20.5, 128^3 (88% of the cache) 53.0 + 40.6 and 49.4 +
// 39.5, 112^3 with a varying diagonal 43.1 + 33.2 and 41.6 + 32.0.
inline int pipe_vectors(bool unif) { return unif ? 14 : 17; }
inline bool rows_stay_near(int64_t rows, int variant, bool unif) {
  return variant == RPK_PIPELINED && (double)pipe_vectors(unif) * (double)rows * 8.0 <= 0.9 * kInfinityCacheBytes;
}

// Vectors of one iteration that stay in the Infinity Cache (those it touches,
// less those streamed past it: x, p, r0 and dinv in the standard loop, x and r0
// with a uniform Jacobi vector)
inline int cached_vectors(int variant, bool near, bool far, bool unif) {
  if (variant == RPK_PIPELINED) return near ? pipe_vectors(unif) : far ? 4 : pipe_kept(unif);
  if (variant == RPK_STD) return std_vectors(unif) - (far ? (unif ? 2 : 4) : 0);
  return unif ? nvec_of(variant) : nvec_of(variant) + 2;  // PCG: r, p, d, y, x, dinv (r, p, d, x)
}

template <template <int> class F, typename... Args>
rpk_status by_fpe(int N, Args&&... args) {
  switch (N) {
    case 0: return F<0>::call(args...);
    case 1: return F<1>::call(args...);
    case 2: return F<2>::call(args...);
    case 3: return F<3>::call(args...);
    case 4: return F<4>::call(args...);
    case 8: return F<8>::call(args...);
  }
  return RPK_ERR_ARG;
}

// ---------------------------------------------------------------------------
// Batches of systems (batch.hip; also used by the server)
// ---------------------------------------------------------------------------
struct Plan {
  std::vector<Tile> tiles;  // XCD-interleaved: tile t runs on XCD t % 8
  std::vector<int> G;       // tiles per listed system
};

// Tiles of at most T rows for the listed systems (sizes n); Tile.sys is ids[k]
// (or k when ids is null) and Tile.rec the tile's index inside its system.
// spread: a system may be cut over several XCDs where whole ones leave XCDs idle.
Plan make_plan(const std::vector<int64_t>& n, int T, const std::vector<int>* ids = nullptr, bool spread = true);
// upper bound of make_plan(n, T).tiles.size() for every T >= Tcap
int64_t tile_capacity(const std::vector<int64_t>& n, int Tcap);

// Device block of one system: tickets + flags | long accumulators | plain-mode
// sums of gcap tiles | nvec solver vectors of n doubles.
// Counters, flags and one counter for each copy of the accumulators (Red), of a
// single call and of a system of a batch (which has one copy and draws no such ticket)
constexpr size_t kTicketBytes = (kSubTickets + kMaxCopies) * sizeof(unsigned);
constexpr size_t kFlagsBytes = 8 * sizeof(unsigned) + MAX_DOTS * sizeof(int);
static_assert(kSubTickets * sizeof(unsigned) == kFlagsBytes, "the copies' counters lie behind the flags");
size_t sys_bytes(int64_t n, int gcap, int nvec);
// Descriptor of a system whose block starts at `base` (device address).
SysDesc make_desc(const rpk_matrix* A, const double* b, double* x, char* base, int gcap, int G, int variant,
                  State* st, double* hist);

// Library-wide state, guarded by g_mu: the capture stream, pinned state
// buffers, and the cache of instantiated iteration graphs.  A graph key lists
// every kernel argument the graph bakes in; key[0] is the matrix handle the
// graph refers to (0 when its kernels find their systems through device memory).
std::mutex& lib_mutex();
hipStream_t capture_stream();
rpk_status ensure_globals();
// pinned host buffer of at least `count` States (valid until the next call)
State* pinned_states(size_t count);
hipGraphExec_t graph_find(const std::vector<uint64_t>& key);
void graph_put(const std::vector<uint64_t>& key, hipGraphExec_t g);
void graph_drop_owner(uint64_t owner);

// Capture `body(capture_stream)` into a graph and instantiate it (cached by key).
template <class Body>
rpk_status graph_get(const std::vector<uint64_t>& key, Body body, hipGraphExec_t* out) {
  hipGraphExec_t exec = graph_find(key);
  if (!exec) {
    hipGraph_t graph = nullptr;
    hipStream_t cs = capture_stream();
    HIPCHK(hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
    const rpk_status cst = body(cs);
    const hipError_t ec = hipStreamEndCapture(cs, &graph);
    if (cst != RPK_OK || ec != hipSuccess) {
      if (graph) (void)hipGraphDestroy(graph);
      return RPK_ERR_HIP;
    }
    const hipError_t ei = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (ei != hipSuccess) return RPK_ERR_HIP;
    graph_put(key, exec);
  }
  *out = exec;
  return RPK_OK;
}

}  // namespace rpkhost
