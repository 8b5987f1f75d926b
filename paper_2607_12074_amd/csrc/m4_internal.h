// m4_internal.h -- shared declarations of the MI355X motif-count library.
// Device arrays of a graph prepared in "rank space": vertices are relabelled
// by the degree order (d, id) (the canonical order of Section III-D), every
// row is sorted, and the oriented out-list N+(r) of vertex r is the suffix of
// its row holding the neighbours of higher rank.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <functional>
#include <string>

#include "../../include/m4.h"

namespace m4 {

constexpr int WAVE = 64;
// the MI355X's last-level cache (Infinity Cache) in front of HBM
constexpr size_t kInfinityCacheBytes = size_t(256) << 20;

// 128-bit unsigned accumulator in device memory, added to with two 64-bit
// atomics (exact: the carry of the low word is derived from its own old value).
struct U128 {
  unsigned long long lo, hi;
};

enum Acc { ACC_K4 = 0, ACC_C4, ACC_S, ACC_P, ACC_PAW2, ACC_D, ACC_SUMT, ACC_N };
// adjacent pairs of A_e x B_e over all edges (edge-anchor basis), in the
// spare accumulator
constexpr int ACC_Z = ACC_N;
// ST_COST to ST_COST + 2: the anchor-selection inputs (wedge endpoints bound,
// edge-basis row entries, longest row)
enum Stat { ST_STEPS = 0, ST_WEDGES, ST_LOOKUPS, ST_HITS, ST_COST, ST_N = 8 };

// 4-cycle-owner buckets by wedge bound.
enum C4Bucket { CB_NONE = 0, CB_TINY, CB_HASH, CB_MED, CB_WIN, CB_BIN, CB_WIDE, CB_N };
// radix digits of the 4-cycle bucket keys and slots of their bucket starts
constexpr int C4_KEY_BITS = 4;
constexpr int C4_START_SLOTS = (1 << C4_KEY_BITS) + 1;

// Largest out-degree handled with the bitmap rows in LDS.
constexpr int TRI_LDS_MAX = 1024;
// 4-cycle window: 32768 words (128 KiB of LDS) of zoned counters.
constexpr int C4_WIN_WORDS = 32768;
constexpr int C4_TINY_MAX = 256;      // tiny owners: one wavefront, a table of twice the bound
constexpr int C4_LIGHT_MAX = 2048;    // largest wedge bound of the light bucket
constexpr int C4_MED_CAP = 12288;     // ... of the medium bucket's first rule
constexpr int C4_MED_MAX = 65536;     // ... of the medium bucket
// Entries of slack after the last row of a rank-space CSR, so that 16-byte
// vector loads aligned below a cursor may run past the end of the array.
constexpr int NCOL_PAD = 256;

// Error bits of Scal::err
constexpr int ERR_INVALID = 1;  // malformed CSR (M4_VALIDATE)
constexpr int ERR_RANGES = 2;   // ranged 4-cycle plan exceeded its bound
constexpr int ERR_PROBE = 4;    // an open-addressing probe ran past its table size

// Stripes of the accumulators: atomics on one address complete one after the
// other (about 14 ns each on the MI355X, whatever adds them), so each
// workgroup adds into the 128-byte stripe its index picks, and the stripes
// are summed at the end.
constexpr int ACC_STRIPES = 32;

// Graphs of at most this many vertices are prepared and planned by three
// kernels and one read-back (m4_small.hip).
constexpr int SMALL_N = 8192;
struct SmallInfo {
  int64_t tri_start[17];
  int64_t c4_start[C4_START_SLOTS + 2];  // bucket starts, then the two zone bounds
  int64_t bound[16];                     // Classes::bound
  unsigned long long cost[4];  // wedge endpoints, bound of the row entries the edge basis
                               // scans, longest row, those row entries
  int64_t hub_slots;
  unsigned int kmax;  // largest out-degree beyond TRI_LDS_MAX, 0 if none
  int dmax;
};

struct Scal {
  unsigned long long stat[ST_N];
  unsigned int dmax;
  int err;
  unsigned int work[8];     // owner counters of the triangle stage
  unsigned int work_c4[8];  // ... of the 4-cycle stage (the stages may overlap)
  unsigned int nhub;  // vertices with a hub table (triangle stage)
  unsigned int pad2;
  unsigned long long out[6];
  unsigned long long basis[8];  // T, K4, C4_ni, S, P_ni, Paw_ni, D_ni, sum_t
  unsigned long long kstat[M4_NK][4];  // per kernel slot: elems, rows, aux, aux2
  int status;
  int pad;
  SmallInfo small;
  alignas(128) U128 acc[ACC_STRIPES][ACC_N + 1];  // not read back to the host
};
constexpr size_t kScalHead = offsetof(Scal, acc);

struct Prep {
  int64_t n = 0, nnz = 0, m = 0;
  int32_t* perm = nullptr;  // rank -> input id
  int32_t* rank = nullptr;  // input id -> rank
  int32_t* dr = nullptr;    // degree by rank (non-decreasing)
  int32_t* dlo = nullptr;   // neighbours of lower rank
  int32_t* dplus = nullptr; // neighbours of higher rank = |N+(r)|
  int64_t* nptr = nullptr;  // row offsets in rank space [n+1]
  int64_t* optr = nullptr;  // oriented edge offsets [n+1]
  int32_t* ncol = nullptr;  // rows in rank space, sorted [nnz]
  uint32_t* t = nullptr;    // triangles per oriented edge [m]
  // Partitioned runs: only owners in [own_lo, own_hi) are processed and rows
  // may be stored as a prefix of row_len[v] entries (null: full rows).
  int64_t own_lo = 0, own_hi = -1;
  const int32_t* row_len = nullptr;
  int64_t hi() const { return own_hi < 0 ? n : own_hi; }
};

// Rank boundaries of degree classes, read back once per graph.
struct Classes {
  int64_t r1;            // first rank with degree >= 2
  int64_t bound[16];     // first rank with degree > thr[i]
  int dmax;
};

// ------------------------------------------------------------ workspace
struct Arena {
  char* base = nullptr;
  size_t cap = 0, used = 0;
  template <typename T>
  T* take(size_t count) {
    size_t bytes = (count * sizeof(T) + 255) & ~size_t(255);
    if (bytes == 0) bytes = 256;
    if (used + bytes > cap) return nullptr;
    T* p = reinterpret_cast<T*>(base + used);
    used += bytes;
    return p;
  }
};

struct Tuning {
  int tri_wave_max = 64;    // <= WAVE
  int c4_light_max = 2048;  // wedge bound for the hash bucket
  int c4_med_max = 12288;   // wedge bound for the one-pass medium hash (0: no medium bucket)
  int batch_variant = 0;    // batched kernel: 0 = 1024 threads / 96 KiB, 1 = 512 / 40 KiB
  int batch_light = 128;    // batched kernel: wedge bound of the wavefront hash
  int hub_min = 128;        // out-degree from which a vertex gets a hub table (0: none)
  int probe_w = 16;         // weight of a hub-table probe against a scanned element (x 1/3)
  int c4_med_win = 64;      // ranged medium owners: 16 windows >= this per range (0: none)
  int c4_bin_win = 6;       // owners above the one-pass medium bound whose endpoints span at
                            // least this many counter windows take the large filter (0: never)
  int c4_bin_cap = 0;       // candidates one class of a large filtered owner is planned for
                            // (0, or more than its table holds: 3/4 of that)
  int c4_bin_dense = 16384; // endpoints per window from which an owner keeps dense windows (0: never)
  int probe_w_far = 64;     // probe_w when the hub tables do not fit in the Infinity Cache
  int tri_wave_far = 64;    // tri_wave_max when the out-lists do not fit in the Infinity Cache
  // weights of the anchor-selection objective, from stage times measured on
  // the MI355X over graphs of 10^2 to 10^7 edges: ns per wedge endpoint
  // bound, fixed us of the wedge stage (what it takes beyond the edge stage
  // when neither has work); ns per row entry the edge basis
  // scans, per owner (the work counter they are taken from serves one in
  // 12 ns) and per entry of the longest row (one thread scans it alone)
  double cost_wedge_ns = 0.005, cost_wedge_fixed_us = 15.0, cost_edge_ns = 0.03;
  double cost_edge_owner_ns = 12.0, cost_edge_row_ns = 1000.0;
};

// Optional per-launch HIP event pairs (M4_TIMING).
struct KTimer {
  bool on = false;
  hipEvent_t ev[M4_NK][2] = {};
  bool used[M4_NK] = {};
  void begin(int k, hipStream_t s) {
    if (on) {
      (void)hipEventRecord(ev[k][0], s);
      used[k] = true;
    }
  }
  void end(int k, hipStream_t s) {
    if (on) (void)hipEventRecord(ev[k][1], s);
  }
};

// ------------------------------------------------------ launch helpers
struct Err {
  int code = M4_OK;
  std::string msg;
};

#define M4_HIP(expr)                                                       \
  do {                                                                     \
    hipError_t e_ = (expr);                                                \
    if (e_ != hipSuccess) {                                                \
      throw ::m4::HipFail(e_, #expr, __FILE__, __LINE__);                  \
    }                                                                      \
  } while (0)

struct HipFail {
  hipError_t e;
  const char* what;
  const char* file;
  int line;
  HipFail(hipError_t e_, const char* w, const char* f, int l) : e(e_), what(w), file(f), line(l) {}
};

struct Fail {
  int code;
  std::string msg;
  Fail(int c, std::string m) : code(c), msg(std::move(m)) {}
};

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ------------------------------------------------- primitives (m4_prims)
// Exclusive scan: out[0..count] with out[count] = total.  tmp must hold
// scan_tmp_elems(count) int64.
size_t scan_tmp_elems(int64_t count);
void scan_i32(const int32_t* in, int64_t count, int64_t* out, int64_t* tmp, hipStream_t s);
void scan_i64(const int64_t* in, int64_t count, int64_t* out, int64_t* tmp, hipStream_t s);

// Stable partition of items [0, count) by a small key (bucket id < 2^bits),
// and the general stable radix pass used by the degree sort.
size_t radix_tmp_elems(int64_t count, int bits);
void radix_pass(const uint32_t* keys_in, const int32_t* vals_in, int64_t count, int shift,
                int bits, uint32_t* keys_out, int32_t* vals_out, int64_t* tmp,
                int64_t* bucket_start /* nullable, [2^bits + 1] */, hipStream_t s,
                int32_t* place = nullptr /* position of every value */);

void fill_u32(void* p, uint32_t v, size_t count32, hipStream_t s);

// --------------------------------------------------- stages (per file)
// m4_build.hip
size_t build_tmp_bytes(int64_t n, int64_t nnz);
void build_prep(const int64_t* rp, const int32_t* col, int64_t n, int64_t nnz, bool validate,
                Prep& P, Classes& C, Scal* scal, Scal* scal_host, Arena& tmp, hipStream_t s);
// Checks a CSR (simple, symmetric, sorted); errors go to scal->err.
void validate_csr(const int64_t* rp, const int32_t* col, int64_t n, int64_t nnz, Scal* scal,
                  hipStream_t s);
// First half of build_prep: degrees, degree order (perm, dr, rank), row
// offsets nptr and the rank boundaries of the degree classes.
void degree_order(const int64_t* rp, const int32_t* col, int64_t n, int64_t nnz, bool validate,
                  Prep& P, Classes& C, Scal* scal, Scal* scal_host, Arena& tmp, hipStream_t s);
void edge_t_to_input(const Prep& P, const int64_t* rp, const int32_t* col, uint32_t* t_out,
                     hipStream_t s);
// Relabels rows [r_lo, r_hi) (ranks) through rank[] and sorts them; per-row
// arrays (perm, nptr, dr, dlo, dplus) are indexed by rank - r_base; bnd are
// the rank boundaries of the degree classes (row_class_thresholds()).
void sort_rows(const int64_t* rp, const int32_t* col, const int32_t* perm, const int32_t* rank,
               const int64_t* nptr, const int32_t* dr, int64_t n, int64_t r_lo, int64_t r_hi,
               const int64_t* bnd, int32_t* ncol, int32_t* dlo, int32_t* dplus, int64_t r_base,
               hipStream_t s);
int row_class_count();
const int* row_class_thresholds();

// An anchor stage is planned on stream s (small kernels and host read-backs
// of bucket sizes) and returns the launches of its heavy kernels, to be
// issued on any stream ordered after s; the stage's workspace and scratch
// stay reserved until those kernels are done.
using Launch = std::function<void(hipStream_t)>;

// m4_tri.hip
// big_scratch(bytes) returns device memory for the hub tables and for owners
// whose bitmap does not fit in LDS (only called when those exist).
// credits, if given, takes the launch that adds the per-vertex credits of the
// owners with out-degree up to 512 (after the count's launch: t complete, the
// workspace and scratch kept) and a bound of the out-degrees if any is larger
// (else 0).
struct TriCredits {
  int kmax = 0;
  std::function<void(hipStream_t, unsigned long long* n12, unsigned long long* n14)> launch;
};
// A stage's plan: its enqueue() buckets the owners (its workspace) and counts
// them (scal->small); once the host has that back, its plan() makes the
// launches.  Both stages share the read-back; graphs of up to SMALL_N vertices
// are planned by small_prep() instead of the enqueues.
struct TriWork {
  uint32_t* key;
  int32_t* order;
  int64_t* rtmp;
  int64_t* hoff64;  // resident runs: hub table offsets, then the out-list records
  int32_t* hoff;    // hub tables (null: none)
  int32_t* hub_list;
  int64_t* hst;
};
TriWork tri_work(const Prep& P, const Tuning& tu, Arena& tmp);
// out-degree bounds of the register kernel (0: unused) and the wavefront kernel
void tri_bounds(const Prep& P, const Tuning& tu, uint32_t flags, uint32_t cache_rows,
                int* small_max, int* wave_max);
void tri_enqueue(const Prep& P, Scal* scal, const Tuning& tu, uint32_t flags, uint32_t cache_rows,
                 const TriWork& w, hipStream_t s);
Launch tri_plan(const Prep& P, Scal* scal, const Tuning& tu, uint32_t flags, uint32_t cache_rows,
                const TriWork& w, int num_cu, const std::function<char*(size_t)>& big_scratch,
                KTimer* kt, const SmallInfo& si, TriCredits* credits = nullptr);
// the counters of the enqueued plans
inline SmallInfo read_plan(const Scal* scal, hipStream_t s) {
  SmallInfo si;
  M4_HIP(hipMemcpyAsync(&si, &scal->small, sizeof(si), hipMemcpyDeviceToHost, s));
  M4_HIP(hipStreamSynchronize(s));
  return si;
}
inline void tri_run(const Prep& P, Scal* scal, const Tuning& tu, uint32_t flags,
                    uint32_t cache_rows, Arena& tmp, hipStream_t s, int num_cu,
                    const std::function<char*(size_t)>& big_scratch) {
  const TriWork w = tri_work(P, tu, tmp);
  tri_enqueue(P, scal, tu, flags, cache_rows, w, s);
  tri_plan(P, scal, tu, flags, cache_rows, w, num_cu, big_scratch, nullptr, read_plan(scal, s))(s);
}

// m4_local.hip: per-vertex orbit counts of a prepared graph (t complete)
void local_orbits(const Prep& P, const Classes& C, Scal* scal, unsigned long long* arrays,
                  const Launch& cycles, const TriCredits& credits, unsigned long long* gscr,
                  int gblocks, unsigned long long* out, int num_cu, hipStream_t s);
size_t local_glob_stride_words(int kmax);

// m4_edge.hip: the cycle/path anchor basis chosen by the anchor-selection
// objective (estimates in ns; edge = adjacent pairs of A_e x B_e)
struct BasisChoice {
  bool edge = false;
  bool pending = false;  // settled without the estimates: basis_costs() fills them in
  double cost_wedge = 0, cost_edge = 0;
};
// in[3]: the objective's inputs, read back where the choice needs them; costs:
// the estimates are wanted (in scal's stat[], if pending)
BasisChoice choose_basis(const Prep& P, const Tuning& tu, uint32_t flags, bool budgeted,
                         bool costs, Scal* scal, unsigned long long* in, hipStream_t s, const SmallInfo* si);
void basis_costs(BasisChoice& b, const Tuning& tu, int64_t n, bool budgeted,
                 const unsigned long long* in);
Launch edge_plan(const Prep& P, Scal* scal, uint32_t flags, int num_cu, KTimer* kt);

// m4_c4.hip (binned, if given, is set when owners go to the large filter,
// which holds every CU with a persistent workgroup and all of its LDS; n8, if
// given, receives the per-vertex 4-cycle credits of every rank, which the
// enqueue has to know of: credit)
struct C4Work {
  int2* wub;  // {wedge bound, lower neighbours of degree above 1}
  uint32_t* key;
  int32_t* order;
  int64_t* rtmp;
  int32_t* hlen;
  int64_t* hoff;
  int64_t* stmp;
  int4* vmeta;  // per-row records of full rows (a partition stores row prefixes instead)
};
C4Work c4_work(const Prep& P, Arena& tmp);
void c4_enqueue(const Prep& P, const Classes& C, Scal* scal, const Tuning& tu, const C4Work& w,
                hipStream_t s, bool credit, KTimer* kt);
Launch c4_plan(const Prep& P, const Classes& C, Scal* scal, const Tuning& tu, uint32_t flags,
               const C4Work& w, hipStream_t s, int num_cu, KTimer* kt,
               const std::function<char*(size_t)>& big_scratch, const SmallInfo& si,
               bool* binned = nullptr, unsigned long long* n8 = nullptr);
inline void c4_run(const Prep& P, const Classes& C, Scal* scal, const Tuning& tu, uint32_t flags,
                   Arena& tmp, hipStream_t s, int num_cu,
                   const std::function<char*(size_t)>& big_scratch) {
  const C4Work w = c4_work(P, tmp);
  c4_enqueue(P, C, scal, tu, w, s, false, nullptr);
  c4_plan(P, C, scal, tu, flags, w, s, num_cu, nullptr, big_scratch, read_plan(scal, s))(s);
}

// m4_small.hip: build_prep, the anchor objective's inputs and the plans of both
// anchor stages for a graph of at most SMALL_N vertices; clears scal and t.
// The host's copy of SmallInfo is scal_host->small afterwards.
void small_prep(const int64_t* rp, const int32_t* col, int64_t n, int64_t nnz, Prep& P, Classes& C,
                const Tuning& tu, uint32_t flags, uint32_t cache_rows, bool credit,
                const TriWork& tw, const C4Work& cw, Scal* scal, Scal* scal_host, hipStream_t s);

// m4_closure.hip
void closure_run(const Prep& P, Scal* scal, uint32_t flags, hipStream_t s);
// zbasis: the 4-cycle statistic is Z of the edge-anchor basis, not C4_ni
void finalize_run(Scal* scal, hipStream_t s, bool zbasis = false);

}  // namespace m4
