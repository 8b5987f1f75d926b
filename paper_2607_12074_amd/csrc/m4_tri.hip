// m4_tri.hip -- triangle and 4-clique anchors (per-edge t_e, K4).
//
// Owner rule: a triangle u<v<w and a 4-clique u<v<w<x (rank order) belong to
// their lowest vertex u.  For an owner u with out-list a = N+(u) (k entries,
// sorted) the kernel builds the induced subgraph of G on a as k bitmap rows:
// bit p of row i is set iff a[p] is in N+(a[i]).  Row i is the candidate
// frontier C(u, a[i]) = N+(u) & N+(a[i]) of the partial embedding (u, a[i]):
// every set bit is a triangle (u, a[i], a[p]), and the frontier is reused by
// every triangle that extends it to a 4-clique, |C(u,a[i]) & C(u,a[p])|
// (induced-signature reuse, Section III-C; the stored state has j = 2 and
// requires adjacency to both embedded vertices, no non-adjacency).
//
// Rows are filled by ordered set intersection (Section III-D): every element
// x of N+(a[i]) is looked up among a[i+1..k).  Owners are split by k: a quarter
// wavefront with everything in registers (k <= 16), one wavefront (k <= 64, one
// 64-bit word per row), one workgroup with the bitmap in LDS (k <= 1024), or
// one workgroup with the bitmap in global scratch (larger k).  Block-local sums
// are folded into one 128-bit atomic per workgroup (block-local aggregation).
#include <limits.h>

#include <algorithm>
#include <array>
#include <type_traits>

#include "m4_plan_dev.h"
#include "m4_tri_dev.h"
#include "m4_walk_dev.h"

namespace m4 {

namespace {

// Owners with the bitmap in LDS, NT threads each.  The rows are resolved in two
// ways, as in tri_owner: rows whose head has a hub table by probing it for the
// later a's, the others by reading their lists.  Few of the read elements are
// among the a's, so a walk only tests them against a bitmap of the a's in LDS
// (bit x mod 2^13) and stops beyond the last a; the ones that pass are gathered
// per wavefront and looked up 64 at a time, instead of probing an LDS table
// for every element.  That table had the kernel bound by the scalar unit (lane
// masks of the probe loops) and by latency; scale-24 web graph, ms: 12.3 M
// owners of out-degree up to 64 (with k_tri_small) 52 -> 29, 0.9 M up to 128
// 34 -> 9.2; with reads this cheap the hub tables pay from out-degree 128 (from
// 32 before: their making 7.3 -> 0.35 ms).  Threads for out-degrees up to 128:
// 64 / 128 / 256 take 8.9 / 9.2 / 11.8 ms there and 1.00 / 0.68 / 0.79 ms on
// the web 2^21 graph; filters of 128 / 512 words instead of 256: +3 / -1 %.
// CRED (orbit counts, t complete): nothing is counted; every triangle gives its
// three vertices the triangles of their opposite edge less one (c12, with tu
// the triangles of the owner's edges), and the bitmap is made symmetric, so
// that the 4-cliques of the owner and a[i] are half the adjacent pairs among
// the neighbours of a[i] (c14), without an atomic per 4-clique.
constexpr int TRI_FILTER_WORDS = 256;

template <int KMAX, int NT, bool CRED>
struct TriShared {
  static constexpr int W = (KMAX + 63) / 64;
  uint64_t B[KMAX * W];
  unsigned long long c12[CRED ? KMAX : 1], c14[CRED ? KMAX : 1];
  int32_t a[KMAX], sst[KMAX + 1], soe[KMAX], slen[KMAX + 1], spref[KMAX + 1];
  uint32_t colcnt[KMAX];    // CRED: the triangles of the owner's edges
  int32_t hp[2 * KMAX];     // positions of the a's by hash; signature tags afterwards
  uint32_t filter[TRI_FILTER_WORDS];
  int16_t scan[KMAX + 1];   // rows that are read
  int32_t qat[NT / WAVE][2 * WAVE];  // per wavefront: places of elements to look up
  int16_t qrow[NT / WAVE][2 * WAVE];  // ... and their rows
  unsigned long long work[4];  // of all owners: steps, looks, hits, words read
  int next, nscan, item;
};

// One thread's sums.  Over all of its owners: k4 (fewer than 2^44 triangles on
// 2^30 edges, each with fewer than 2^9 common bits), escan, ksum (at most the
// edges) and owners (at most the vertices).  Of one owner, added to the
// workgroup's 64-bit counters after it: steps and looks are at most its 512 rows
// of fewer than 2^16 entries, wread about twice that.  (In 64-bit registers over
// all owners they made the kernels spill 60 to 76 bytes a lane.)
struct TriCounts {
  unsigned long long k4 = 0, escan = 0;
  uint32_t ksum = 0, owners = 0;
  uint32_t steps = 0, looks = 0, hits = 0, wread = 0;
};

template <int KMAX, int NT, bool CRED>
__device__ __forceinline__ void tri_owner_lds(const TriArgs& A, int32_t u,
                                              TriShared<KMAX, NT, CRED>& S, TriCounts& C) {
  const int tid = threadIdx.x, lane = tid & (WAVE - 1);
  const OutList lu = out_list(A, u);
  const int k = __builtin_amdgcn_readfirstlane(lu.len);
  const int64_t rb = lu.st, oe_u = lu.oe;
  const int W = (k + 63) >> 6;
  int H = 16, hshift = 28;
  while (H < 2 * k) {
    H <<= 1;
    hshift--;
  }
  C.ksum += (uint32_t)k;  // the same in every thread
  C.owners++;
  if (tid == 0) {
    S.next = S.nscan = 0;
    // the empty segment after the last scanned row
    S.sst[KMAX] = S.slen[KMAX] = 0;
  }
  for (int i = tid; i < k * W; i += NT) S.B[i] = 0;
  for (int i = tid; i < H; i += NT) S.hp[i] = -1;
  for (int i = tid; i < TRI_FILTER_WORDS; i += NT) S.filter[i] = 0;
  __syncthreads();
  for (int i = tid; i < k; i += NT) {
    const int32_t v = A.ncol[rb + i];
    S.a[i] = v;
    const OutList lv = out_list(A, v);
    const int L = lv.len;
    int32_t st = lv.st;
    if (A.hub_min > 0 && L >= A.hub_min && A.probe_w * (k - 1 - i) < 3 * L) {
      const int32_t off = A.hoff[v];
      if (off >= 0) st = -1 - off;  // probe row: table offset, negated
    }
    S.sst[i] = st;
    S.soe[i] = lv.oe;
    S.slen[i] = L;
    C.escan += (unsigned long long)L;
    // the last row has no later entries
    if (st >= 0 && L > 0 && i + 1 < k) S.scan[atomicAdd(&S.nscan, 1)] = (int16_t)i;
    if (CRED) {
      S.colcnt[i] = A.t[oe_u + i];
      S.c12[i] = S.c14[i] = 0;
    } else {
      S.colcnt[i] = 0;
    }
    atomicOr(&S.filter[((uint32_t)v >> 5) & (TRI_FILTER_WORDS - 1)], 1u << (v & 31));
    // k distinct keys in H >= 2k slots: a free slot is met within H probes
    uint32_t h = ((uint32_t)v * 0x9E3779B1u) >> hshift;
    int probes = 0;
    while (atomicCAS(&S.hp[h], -1, i) != -1) {
      h = (h + 1) & (uint32_t)(H - 1);
      if (++probes >= H) {
        atomicOr(A.err, ERR_PROBE);
        break;
      }
    }
  }
  __syncthreads();
  // exclusive prefix of the probes of a[0..k) into spref[0..k]
  {
    const int per = (k + NT - 1) / NT;
    const int lo = tid * per;
    int64_t s = 0;
    for (int i = lo; i < lo + per && i < k; i++) s += S.sst[i] < 0 ? k - 1 - i : 0;
    int64_t tot;
    int64_t run = block_excl_scan64<NT>(s, &tot);
    for (int i = lo; i < lo + per && i < k; i++) {
      S.spref[i] = (int32_t)run;
      run += S.sst[i] < 0 ? k - 1 - i : 0;
    }
    if (tid == 0) {
      S.spref[k] = (int32_t)tot;
      S.scan[S.nscan] = KMAX;
    }
  }
  __syncthreads();
  unsigned long long cu12 = 0;  // CRED: this thread's share of the owner's credit
  // a[p] found in row i, edge e of the oriented edges
  auto found = [&](int i, int p, int32_t e) {
    atomicOr((unsigned long long*)&S.B[i * W + (p >> 6)], 1ull << (p & 63));
    if (CRED) {
      atomicOr((unsigned long long*)&S.B[p * W + (i >> 6)], 1ull << (i & 63));
      cu12 += (unsigned long long)A.t[e] - 1;
      atomicAdd(&S.c12[p], (unsigned long long)S.colcnt[i] - 1);
      atomicAdd(&S.c12[i], (unsigned long long)S.colcnt[p] - 1);
    } else {
      atomicAdd(&S.colcnt[p], 1u);
      atomicAdd(&A.t[e], 1u);
    }
  };
  // ---- scanned rows
  const int nscan = __builtin_amdgcn_readfirstlane(S.nscan);
  if (nscan > 0) {
    const int32_t hi = S.a[k - 1] + 1;
    int32_t* qat = S.qat[tid / WAVE];
    int16_t* qrow = S.qrow[tid / WAVE];
    int qn = 0;  // uniform in the wavefront
    auto look_up = [&](int m) {
      wave_sync();
      if (lane < m) {
        const int32_t at = qat[qn - m + lane];
        const int i = qrow[qn - m + lane];
        const int32_t x = A.ncol[at];
        uint32_t h = ((uint32_t)x * 0x9E3779B1u) >> hshift;
        int p = -1;
        for (int probes = 0; probes <= H; probes++) {
          p = S.hp[h];
          if (p < 0 || S.a[p] == x) break;
          h = (h + 1) & (uint32_t)(H - 1);
        }
        if (p >= 0) found(i, p, S.soe[i] + (at - S.sst[i]));
      }
      qn -= m;
      wave_sync();
    };
    unsigned read = 0;
    seg_walk<8>(
        A.ncol, hi, nscan, &S.next,
        [&](int j) {
          const int i = S.scan[j];
          const int32_t st = S.sst[i];
          return make_int2(st, st + S.slen[i]);
        },
        [&](const int32_t(&x)[4], int j, int at) {
          const int i = S.scan[j];
#pragma unroll
          for (int q = 0; q < 4; q++) {
            const bool in = x[q] < hi;
            read += in;
            const bool is =
                in && ((S.filter[((uint32_t)x[q] >> 5) & (TRI_FILTER_WORDS - 1)] >> (x[q] & 31)) & 1);
            const uint64_t m = __ballot(is);
            if (is) {
              const int w = qn + lanes_before(m);
              qat[w] = at + q;
              qrow[w] = (int16_t)i;
            }
            qn += __popcll(m);
            if (qn >= WAVE) look_up(WAVE);
          }
        },
        [](int, bool) {});
    if (qn > 0) look_up(qn);
    C.steps += read;
    C.wread += read;
  }
  // ---- probed rows: (row, later a) pairs dealt to the threads, the first
  // slots of four pairs read before they are compared
  const int total = __builtin_amdgcn_readfirstlane(S.spref[k]);
  if (total > 0) {
    int i = tid < total ? upper_index(S.spref, k, tid) : 0;
    int ii[4], pp[4];
    unsigned long long ee[4];
    auto fetch = [&](int q0) {
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int q = q0 + r * NT;
        ii[r] = -1;
        if (q < total) {
          while (S.spref[i + 1] <= q) i++;
          ii[r] = i;
          pp[r] = i + 1 + q - S.spref[i];
          ee[r] = A.htab[(int64_t)(-1 - S.sst[i]) + hub_hash(S.a[pp[r]], hub_bits(S.slen[i]))];
        }
      }
    };
    fetch(tid);
    for (int q0 = tid; q0 < total; q0 += 4 * NT) {
      int ci[4], cp[4];
      unsigned long long ce[4];
#pragma unroll
      for (int r = 0; r < 4; r++) {
        ci[r] = ii[r];
        cp[r] = pp[r];
        ce[r] = ee[r];
      }
      if (q0 + 4 * NT < total) fetch(q0 + 4 * NT);
#pragma unroll
      for (int r = 0; r < 4; r++) {
        if (ci[r] < 0) continue;
        const int32_t x = S.a[cp[r]];
        const int64_t off = -1 - (int64_t)S.sst[ci[r]];
        const int bits = hub_bits(S.slen[ci[r]]);
        const uint32_t mask = (1u << bits) - 1u;
        uint32_t h = hub_hash(x, bits);
        unsigned long long e = ce[r];
        int pos = -1;
        C.steps++;
        C.wread += 2;
        // load <= 1/2: an empty slot ends every probe within mask + 1 steps
        for (uint32_t probes = 0; e != HUB_EMPTY; probes++) {
          if ((int32_t)(e >> 32) == x) {
            pos = (int)(uint32_t)e;
            break;
          }
          if (probes >= mask) {
            atomicOr(A.err, ERR_PROBE);
            break;
          }
          h = (h + 1) & mask;
          e = A.htab[off + h];
          C.wread += 2;
        }
        if (pos >= 0) found(ci[r], cp[r], S.soe[ci[r]] + pos);
      }
    }
  }
  __syncthreads();
  if (CRED) {
    unsigned long long cu14 = 0;
    for (int q = tid; q < k * W; q += NT) {
      const int i = W == 1 ? q : q / W;
      uint64_t bits = S.B[q];
      unsigned long long c = 0;
      while (bits) {
        const int p = ((q - i * W) << 6) + __ffsll((long long)bits) - 1;
        bits &= bits - 1;
        for (int w = 0; w < W; w++) c += __popcll(S.B[i * W + w] & S.B[p * W + w]);
      }
      if (c) atomicAdd(&S.c14[i], c);
      cu14 += c;
    }
    __syncthreads();
    for (int i = tid; i < k; i += NT) {
      if (S.c12[i]) atomicAdd(&A.n12[S.a[i]], S.c12[i]);
      if (S.c14[i]) atomicAdd(&A.n14[S.a[i]], S.c14[i] / 2);
    }
    // each 4-clique with the owner was met six times
    int64_t tot;
    block_excl_scan64<NT>((int64_t)cu12, &tot);
    if (tid == 0 && tot) atomicAdd(&A.n12[u], (unsigned long long)tot);
    block_excl_scan64<NT>((int64_t)cu14, &tot);
    if (tid == 0 && tot) atomicAdd(&A.n14[u], (unsigned long long)tot / 6);
    __syncthreads();
    return;
  }
  // triangles on the owner's own out-edges: (u, a[i], *) and (u, *, a[i]).  The
  // rows that fit the cache capacity are published with their signature (j = 2,
  // slot i, adjacency to both embedded vertices required, no non-adjacency);
  // other rows stay unpublished and are recomputed.
  uint32_t* tag = reinterpret_cast<uint32_t*>(S.hp);
  const bool cache_on = !(A.flags & M4_NO_CACHE);
  const uint32_t cap = A.cache_rows ? A.cache_rows : 0xffffffffu;
  for (int i = tid; i < k; i += NT) {
    uint32_t c = S.colcnt[i];
    for (int w = 0; w < W; w++) c += __popcll(S.B[i * W + w]);
    if (c) atomicAdd(&A.t[oe_u + i], c);
    tag[i] = (cache_on && (uint32_t)i < cap) ? sig_key(2, (uint32_t)i, 3, 0) : 0u;
  }
  __syncthreads();
  // 4-cliques: for every triangle (u, a[i], a[p]) intersect the two frontiers.
  // A thread takes a row, or a word of one where that still leaves threads
  // idle (k up to half of them: <128, 256> 2 % faster, <512, 256> 13 % slower
  // by words)
  const bool words = 2 * k <= NT;
  for (int q = tid; q < (words ? k * W : k); q += NT) {
    const int i = words ? (W == 1 ? q : q / W) : q;
    const int w0 = words ? q - i * W : 0, w1 = words ? w0 + 1 : W;
    const bool ci = tag[i] == sig_key(2, (uint32_t)i, 3, 0);
    for (int w = w0; w < w1; w++) {
      uint64_t bits = S.B[i * W + w];
      while (bits) {
        const int p = (w << 6) + __ffsll((long long)bits) - 1;
        bits &= bits - 1;
        C.looks++;
        if (ci && tag[p] == sig_key(2, (uint32_t)p, 3, 0)) {
          C.hits++;
          uint64_t c = 0;
          for (int ww = p >> 6; ww < W; ww++)
            c += __popcll(S.B[i * W + ww] & S.B[p * W + ww]);
          C.k4 += c;
        } else {
          // probed rows keep a table offset in sst[]: take the list start again
          const int64_t si = S.sst[i] < 0 ? out_list(A, S.a[i]).st : S.sst[i];
          const int64_t sp = S.sst[p] < 0 ? out_list(A, S.a[p]).st : S.sst[p];
          C.k4 += k4_recompute(A.ncol, S.a, k, p, si, S.slen[i], sp, S.slen[p]);
        }
      }
    }
  }
  __syncthreads();
}

struct TriCounts64 {
  u128_t k4 = 0;
  unsigned long long steps = 0, looks = 0, hits = 0, ksum = 0, wread = 0, escan = 0, owners = 0;
};

template <int NT>
__device__ __forceinline__ void tri_counts_out(const TriArgs& A, const TriCounts64& C) {
  block_add_acc<NT>(A.scal, ACC_K4, C.k4);
  if (A.flags & M4_STATS) {
    block_add_u64<NT>(&A.scal->stat[ST_STEPS], C.steps);
    block_add_u64<NT>(&A.scal->stat[ST_LOOKUPS], C.looks);
    block_add_u64<NT>(&A.scal->stat[ST_HITS], C.hits);
    block_add_u64<NT>(&A.scal->kstat[A.slot][0], C.escan);
    block_add_u64<NT>(&A.scal->kstat[A.slot][1], C.owners);
    block_add_u64<NT>(&A.scal->kstat[A.slot][2], C.ksum);
    block_add_u64<NT>(&A.scal->kstat[A.slot][3], C.wread);
  }
}

// At least 5 wavefronts per SIMD: the register cap hides more of the load and
// probe latency of the owners whose LDS footprint allows it (out-degree up to
// 256); the larger owners are bound by LDS either way.
template <int KMAX, int NT, bool CRED>
__global__ __launch_bounds__(NT, 5) void k_tri_lds(TriArgs A) {
  __shared__ TriShared<KMAX, NT, CRED> S;
  const int64_t b0 = A.start[A.bucket];
  const uint32_t cnt = (uint32_t)(A.start[A.bucket + 1] - b0);
  const int32_t* order = A.order + b0;
  TriCounts C;
  if (threadIdx.x < 4) S.work[threadIdx.x] = 0;
  __syncthreads();
  // runs of A.grab owners from the work counter, or (0) owners dealt in turn
  for (uint32_t turn = blockIdx.x;; turn += gridDim.x) {
    uint32_t first = turn;
    if (A.grab > 0) {
      if (threadIdx.x == 0) S.item = (int)atomicAdd(A.work, (unsigned)A.grab);
      __syncthreads();
      first = (uint32_t)__builtin_amdgcn_readfirstlane(S.item);
      __syncthreads();
    }
    if (first >= cnt) break;
    uint32_t left = A.grab > 0 ? min((uint32_t)A.grab, cnt - first) : 1;
    for (; left > 0; left--, first++) {
      tri_owner_lds<KMAX, NT, CRED>(A, __builtin_amdgcn_readfirstlane(order[first]), S, C);
      if (!CRED) {
        if (A.flags & M4_STATS) {
          const uint32_t of_owner[4] = {C.steps, C.looks, C.hits, C.wread};
          for (int i = 0; i < 4; i++)
            if (of_owner[i]) atomicAdd(&S.work[i], (unsigned long long)of_owner[i]);
        }
        C.steps = C.looks = C.hits = C.wread = 0;
      }
    }
  }
  if (!CRED) {
    TriCounts64 T;
    T.k4 = C.k4;
    T.escan = C.escan;
    __syncthreads();
    if (threadIdx.x == 0) {
      T.ksum = C.ksum;
      T.owners = C.owners;
      T.steps = S.work[0];
      T.looks = S.work[1];
      T.hits = S.work[2];
      T.wread = S.work[3];
    }
    tri_counts_out<NT>(A, T);
  }
}

// Out-degree in (512, 1024]: the bitmap alone nearly fills the LDS.
template <int KMAX, int NT>
__global__ __launch_bounds__(NT) void k_tri_large(TriArgs A) {
  constexpr int WMAX = (KMAX + 63) / 64;
  __shared__ int32_t a[KMAX], sst[KMAX], soe[KMAX], slen[KMAX], spref[KMAX + 1];
  __shared__ uint32_t colcnt[KMAX], tag[KMAX];
  __shared__ uint64_t B[KMAX * WMAX];
  __shared__ int s_item;
  const int64_t b0 = A.start[A.bucket], cnt = A.start[A.bucket + 1] - b0;
  TriCounts64 C;
  for (;;) {
    if (threadIdx.x == 0) s_item = (int)atomicAdd(A.work, 1u);
    __syncthreads();
    const int64_t item = s_item;
    __syncthreads();
    if (item >= cnt) break;
    tri_owner<NT, false, false, true>(A, A.order[b0 + item], threadIdx.x, a, sst, soe, slen, spref,
                                      colcnt, tag, B, C.k4, C.steps, C.looks, C.hits, C.ksum,
                                      C.wread, C.escan);
    if (threadIdx.x == 0) C.owners++;
  }
  tri_counts_out<NT>(A, C);
}

// Owners with out-degree k <= TRI_SMALL: 16 lanes each, four to a wavefront,
// with everything in registers.  Lane i holds a[i], its out-list's record and
// row i of the bitmap; the rows are read one after the other, 16 elements at a
// time (the first reads of four rows go out together), and an element is
// looked up by comparing it with the 16 a's as they rotate through the lanes.
// A wavefront per owner with LDS arrays spent most of its instructions on
// setup here.  A row whose head has a hub table is probed for the later a's,
// one lane each, by the same rule as in the LDS kernels.  Geometric graph of
// 2 M vertices (k about 4.5): 2.4 ms by wavefronts, 0.7 ms so.
constexpr int TRI_SMALL = 16;

template <int N>
__device__ __forceinline__ int row_ror(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xf, 0xf, false);
}
// The rotations of a lane's place in its group, taken once; and the position
// of x among the 16 a's of the group, -1 if none.  Every lane takes part in
// every rotation (none stands under a condition).
struct Rot16 {
  int at[16];
};
__device__ __forceinline__ Rot16 rotations(int i) {
  Rot16 r;
  r.at[0] = i;
#define M4_ROT(N) r.at[N] = row_ror<N>(i);
  M4_ROT(1) M4_ROT(2) M4_ROT(3) M4_ROT(4) M4_ROT(5) M4_ROT(6) M4_ROT(7) M4_ROT(8)
  M4_ROT(9) M4_ROT(10) M4_ROT(11) M4_ROT(12) M4_ROT(13) M4_ROT(14) M4_ROT(15)
#undef M4_ROT
  return r;
}
__device__ __forceinline__ int find16(int x, int a, const Rot16& rot) {
  int p = a == x ? rot.at[0] : -1;
#define M4_ROT(N)                  \
  {                                \
    const int y = row_ror<N>(a);   \
    p = y == x ? rot.at[N] : p;    \
  }
  M4_ROT(1) M4_ROT(2) M4_ROT(3) M4_ROT(4) M4_ROT(5) M4_ROT(6) M4_ROT(7) M4_ROT(8)
  M4_ROT(9) M4_ROT(10) M4_ROT(11) M4_ROT(12) M4_ROT(13) M4_ROT(14) M4_ROT(15)
#undef M4_ROT
  return p;
}
__device__ __forceinline__ uint32_t or16(uint32_t v) {
  v |= (uint32_t)row_ror<8>((int)v);
  v |= (uint32_t)row_ror<4>((int)v);
  v |= (uint32_t)row_ror<2>((int)v);
  v |= (uint32_t)row_ror<1>((int)v);
  return v;
}

template <bool CRED>
__global__ __launch_bounds__(256) void k_tri_small(TriArgs A) {
  constexpr int G = TRI_SMALL, AHEAD = 4;
  const int lane = threadIdx.x & (WAVE - 1), i = lane & (G - 1), gb = lane & ~(G - 1);
  const int64_t b0 = A.start[A.bucket], cnt = A.start[A.bucket + 1] - b0;
  const int64_t waves = (int64_t)gridDim.x * (256 / WAVE);
  const Rot16 rot = rotations(i);
  u128_t k4 = 0;
  unsigned long long steps = 0, looks = 0, ksum = 0, owners = 0, escan = 0;
  for (int64_t base = ((int64_t)blockIdx.x * (256 / WAVE) + threadIdx.x / WAVE) * (WAVE / G);
       base < cnt; base += waves * (WAVE / G)) {
    const int64_t item = base + lane / G;
    const bool valid = item < cnt;
    const int32_t u = valid ? A.order[b0 + item] : 0;
    const OutList lu = valid ? out_list(A, u) : OutList{0, 0, 0};
    const int k = lu.len;
    const bool own = i < k;
    const int32_t a = own ? A.ncol[lu.st + i] : -1 - i;  // no element is negative
    const OutList lv = own ? out_list(A, a) : OutList{0, 0, 0};
    const uint32_t tu = CRED && own ? A.t[lu.oe + i] : 0;
    // table offset of the lane's row where it is probed, else -1
    const int32_t hub = own && A.hub_min > 0 && lv.len >= A.hub_min &&
                                A.probe_w * (k - 1 - i) < 3 * lv.len
                            ? A.hoff[a]
                            : -1;
    int kmax = k;  // over the wavefront's groups
#pragma unroll
    for (int o = WAVE / 2; o >= G; o >>= 1) kmax = max(kmax, __shfl_xor(kmax, o, WAVE));
    uint32_t mask = 0;
    unsigned long long cu12 = 0;
    // a hit of row r: bit p of it, the far edge at position j of its list
    auto found = [&](int r, bool hit, int p, int32_t oe, int j) {
      if (hit) {
        if (CRED) cu12 += (unsigned long long)A.t[oe + j] - 1;
        else atomicAdd(&A.t[oe + j], 1u);
      }
      const uint32_t m = or16(hit ? 1u << p : 0u);
      if (i == r) mask |= m;
    };
    // one step of row r: element x at position j of its list
    auto step = [&](int r, int32_t x, bool in, int32_t oe, int j) {
      const int p = find16(x, a, rot);
      found(r, in && p >= 0, p, oe, j);
      steps += in;
    };
    // the last row has no later entries
    for (int r0 = 0; r0 < kmax - 1; r0 += AHEAD) {
      int32_t st[AHEAD], len[AHEAD], oe[AHEAD], x[AHEAD], tab[AHEAD], bits[AHEAD];
      unsigned long long e[AHEAD];
#pragma unroll
      for (int q = 0; q < AHEAD; q++) {
        const int r = r0 + q;
        st[q] = __shfl(lv.st, gb + (r & (G - 1)), WAVE);
        oe[q] = __shfl(lv.oe, gb + (r & (G - 1)), WAVE);
        len[q] = __shfl(lv.len, gb + (r & (G - 1)), WAVE);
        tab[q] = __shfl(hub, gb + (r & (G - 1)), WAVE);
        bits[q] = 1;
        if (r >= k - 1) len[q] = 0;
        e[q] = HUB_EMPTY;
        if (len[q] == 0) tab[q] = -1;
        if (tab[q] >= 0) {
          bits[q] = hub_bits(len[q]);
          len[q] = 0;  // probed, not scanned
          if (own && i > r) e[q] = A.htab[(int64_t)tab[q] + hub_hash(a, bits[q])];
        }
        x[q] = i < len[q] ? A.ncol[st[q] + i] : INT_MAX;
      }
#pragma unroll
      for (int q = 0; q < AHEAD; q++) {
        if (__ballot(tab[q] >= 0)) {
          // load <= 1/2: an empty slot ends every probe within the table
          const uint32_t hmask = (1u << bits[q]) - 1u;
          uint32_t h = hub_hash(a, bits[q]);
          int pos = -1;
          const bool asked = tab[q] >= 0 && own && i > r0 + q;
          for (uint32_t probes = 0; e[q] != HUB_EMPTY; probes++) {
            if ((int32_t)(e[q] >> 32) == a) {
              pos = (int)(uint32_t)e[q];
              break;
            }
            if (probes >= hmask) {
              atomicOr(A.err, ERR_PROBE);
              break;
            }
            h = (h + 1) & hmask;
            e[q] = A.htab[(int64_t)tab[q] + h];
          }
          found(r0 + q, pos >= 0, i, oe[q], pos);
          steps += asked;
        }
        if (!__ballot(len[q] > 0)) continue;
        step(r0 + q, x[q], i < len[q], oe[q], i);
        for (int j = i + G; __ballot(j - i < len[q]); j += G) {
          const bool in = j < len[q];
          step(r0 + q, in ? A.ncol[st[q] + j] : INT_MAX, in, oe[q], j);
        }
      }
    }
    if (CRED) {
      uint32_t col = 0;
      unsigned long long c12 = 0;
      for (int r = 0; r < kmax; r++) {
        const uint32_t mr = (uint32_t)__shfl((int)mask, gb + r, WAVE);
        const unsigned long long tr =
            (unsigned long long)(uint32_t)__shfl((int)tu, gb + r, WAVE) - 1;
        if ((mr >> i) & 1) {
          col |= 1u << r;
          c12 += tr;
        }
        if ((mask >> r) & 1) c12 += tr;
      }
      const uint32_t adj = mask | col;
      unsigned c14 = 0;  // at most 16 rows of 16 bits
      for (int r = 0; r < kmax; r++) {
        const uint32_t ar = (uint32_t)__shfl((int)adj, gb + r, WAVE);
        if ((adj >> r) & 1) c14 += __popc(ar & adj);
      }
      if (c12) atomicAdd(&A.n12[a], c12);
      if (c14) atomicAdd(&A.n14[a], (unsigned long long)(c14 / 2));
      unsigned long long cu14 = c14;
#pragma unroll
      for (int o = G / 2; o > 0; o >>= 1) {
        cu12 += __shfl_xor(cu12, o, WAVE);
        cu14 += __shfl_xor(cu14, o, WAVE);
      }
      if (i == 0 && cu12) atomicAdd(&A.n12[u], cu12);
      if (i == 0 && cu14) atomicAdd(&A.n14[u], cu14 / 6);
    } else {
      uint32_t c = __popc(mask);  // triangles on the owner's edge to a[i]
      unsigned q4 = 0;  // at most 16 rows of 16 bits
      for (int r = 0; r < kmax; r++) {
        const uint32_t mr = (uint32_t)__shfl((int)mask, gb + r, WAVE);
        if ((mr >> i) & 1) {
          c++;
          looks++;
          q4 += __popc(mr & mask);
        }
      }
      k4 += q4;
      if (own && c) atomicAdd(&A.t[lu.oe + i], c);
    }
    escan += (unsigned long long)lv.len;
    if (i == 0) {
      ksum += (unsigned long long)k;
      owners += valid;
    }
  }
  if (!CRED) {
    block_add_acc<256>(A.scal, ACC_K4, k4);
    if (A.flags & M4_STATS) {
      block_add_u64<256>(&A.scal->stat[ST_STEPS], steps);
      block_add_u64<256>(&A.scal->stat[ST_LOOKUPS], looks);
      block_add_u64<256>(&A.scal->stat[ST_HITS], looks);
      block_add_u64<256>(&A.scal->kstat[A.slot][0], escan);
      block_add_u64<256>(&A.scal->kstat[A.slot][1], owners);
      block_add_u64<256>(&A.scal->kstat[A.slot][2], ksum);
      block_add_u64<256>(&A.scal->kstat[A.slot][3], steps);
    }
  }
}

// Owners whose bitmap does not fit in LDS: the same algorithm over a
// per-block slice of global scratch (atomic loads read past the L1).
template <int NT>
__global__ __launch_bounds__(NT) void k_tri_global(TriArgs A) {
  __shared__ int s_item;
  const int64_t b0 = A.start[A.bucket], cnt = A.start[A.bucket + 1] - b0;
  const int64_t K = A.kmax, WK = (K + 63) / 64;
  uint64_t* B = A.gbits + (int64_t)blockIdx.x * K * WK;
  int32_t* base = A.garr + (int64_t)blockIdx.x * (7 * K + 2);
  int32_t *a = base, *sst = base + K, *soe = base + 2 * K, *slen = base + 3 * K;
  int32_t* spref = base + 4 * K;
  uint32_t* colcnt = (uint32_t*)(base + 5 * K + 1);
  uint32_t* tag = (uint32_t*)(base + 6 * K + 1);
  TriCounts64 C;
  for (;;) {
    if (threadIdx.x == 0) s_item = (int)atomicAdd(A.work, 1u);
    __syncthreads();
    const int64_t item = s_item;
    __syncthreads();
    if (item >= cnt) break;
    tri_owner<NT, true, false, true>(A, A.order[b0 + item], threadIdx.x, a, sst, soe, slen, spref,
                                     colcnt, tag, B, C.k4, C.steps, C.looks, C.hits, C.ksum,
                                     C.wread, C.escan);
    if (threadIdx.x == 0) C.owners++;
    __threadfence();
  }
  tri_counts_out<NT>(A, C);
}

// bucket of every owner by its out-degree k

__global__ void k_tri_keys(const int32_t* __restrict__ dplus, int64_t n, int64_t own_lo,
                           int64_t own_hi, int small_max, int wave_max, uint32_t* __restrict__ key,
                           Scal* scal) {
  int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= n) return;
  int k = (u >= own_lo && u < own_hi) ? dplus[u] : 0;
  const uint32_t b = tri_bucket(k, small_max, wave_max);
  if (b == TK_GLOBAL) atomicMax(&scal->small.kmax, (unsigned int)k);
  key[u] = b;
}

// Hub tables (a vertex with out-degree >= hub_min gets an open-addressing
// table of its out-list, mapping a rank to its position in N+(v)).
__global__ __launch_bounds__(256) void k_hub_size(const int32_t* __restrict__ dplus, int64_t n,
                                                  int hub_min, int32_t* __restrict__ hsz,
                                                  int32_t* __restrict__ hubs, Scal* scal) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int L = v < n ? dplus[v] : 0;
  const bool hub = v < n && L >= hub_min;
  const int slots = hub ? (1 << hub_bits(L)) : 0;
  if (v < n) hsz[v] = slots;
  if (hub) hubs[atomicAdd(&scal->nhub, 1u)] = (int32_t)v;
  block_add_u64<256>(reinterpret_cast<unsigned long long*>(&scal->small.hub_slots),
                     (unsigned long long)slots);
}

__global__ void k_hub_off(const int32_t* __restrict__ hsz, const int64_t* __restrict__ off64,
                          int64_t n, int32_t* __restrict__ hoff) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  hoff[v] = hsz[v] ? (int32_t)off64[v] : -1;
}

// out-list records {start, first oriented edge} of every vertex; the one past
// the last holds the end of the edges
__global__ void k_tri_list(const int64_t* __restrict__ nptr, const int32_t* __restrict__ dlo,
                           const int64_t* __restrict__ optr, int64_t n, int2* __restrict__ list) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v > n) return;
  list[v] = make_int2(v < n ? (int)(nptr[v] + dlo[v]) : 0, (int)optr[v]);
}

// one wavefront per hub (grid-stride over the hub list); lanes insert the
// out-list entries with 64-bit compare-and-swap
__global__ __launch_bounds__(256) void k_hub_insert(const int32_t* __restrict__ dplus,
                                                    const int64_t* __restrict__ nptr,
                                                    const int32_t* __restrict__ dlo,
                                                    const int32_t* __restrict__ ncol,
                                                    const int32_t* __restrict__ hoff,
                                                    const int32_t* __restrict__ hubs,
                                                    const unsigned int* __restrict__ nhub,
                                                    unsigned long long* __restrict__ htab,
                                                    int* __restrict__ err) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t nw = (int64_t)gridDim.x * (blockDim.x / WAVE);
  const int64_t nh = *nhub;
  for (int64_t hix = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE; hix < nh;
       hix += nw) {
    const int32_t v = hubs[hix];
    const int32_t off = hoff[v];
    const int L = dplus[v];
    const int bits = hub_bits(L);
    const uint32_t mask = (1u << bits) - 1u;
    const int64_t st = nptr[v] + dlo[v];
    for (int j = lane; j < L; j += WAVE) {
      const int32_t x = ncol[st + j];
      uint32_t h = hub_hash(x, bits);
      const unsigned long long e = ((unsigned long long)(uint32_t)x << 32) | (uint32_t)j;
      // L distinct keys in 2^bits >= 2L slots: a free slot within 2^bits probes
      for (uint32_t probes = 0;
           atomicCAS(&htab[(int64_t)off + h], HUB_EMPTY, e) != HUB_EMPTY; probes++) {
        if (probes >= mask) {
          atomicOr(err, ERR_PROBE);
          break;
        }
        h = (h + 1) & mask;
      }
    }
  }
}

}  // namespace

// host-side replica of the signature key, for tests of its distinctness
extern "C" uint32_t m4_internal_sig_key(uint32_t j, uint32_t slot, uint32_t mplus, uint32_t mminus) {
  return sig_key(j, slot, mplus, mminus);
}

namespace {
// out-list records and hub tables: resident runs only (a partition holds only
// its halo rows)
inline bool full_rows(const Prep& P) { return P.own_hi < 0 && !P.row_len; }
}  // namespace

TriWork tri_work(const Prep& P, const Tuning& tu, Arena& tmp) {
  const int64_t n = P.n;
  TriWork w{};
  w.key = tmp.take<uint32_t>(n);
  w.order = tmp.take<int32_t>(n);
  w.rtmp = tmp.take<int64_t>(radix_tmp_elems(n, 4));
  if (!w.key || !w.order || !w.rtmp) throw Fail(M4_EINTERNAL, "workspace too small (tri)");
  if (full_rows(P)) {
    w.hoff64 = tmp.take<int64_t>(n + 1);
    if (!w.hoff64) throw Fail(M4_EINTERNAL, "workspace too small (out-lists)");
    if (tu.hub_min > 0) {
      w.hoff = tmp.take<int32_t>(n);
      w.hub_list = tmp.take<int32_t>(n);
      w.hst = tmp.take<int64_t>(scan_tmp_elems(n));
      if (!w.hoff || !w.hub_list || !w.hst) throw Fail(M4_EINTERNAL, "workspace too small (hubs)");
    }
  }
  return w;
}

void tri_bounds(const Prep& P, const Tuning& tu, uint32_t flags, uint32_t cache_rows,
                int* small_max, int* wave_max) {
  // the bound of the owners of one wavefront has one value for out-lists that
  // stream from HBM and one for those in the Infinity Cache (both 64 now)
  const int req = (size_t)P.m * 4 > kInfinityCacheBytes ? tu.tri_wave_far : tu.tri_wave_max;
  *wave_max = req < 2 ? 2 : (req > 64 ? 64 : req);
  // the register kernel holds every frontier, so it is left out where the
  // cache is off or capped below it
  const bool small = !(flags & M4_NO_CACHE) &&
                     (cache_rows == 0 || cache_rows >= (uint32_t)TRI_SMALL);
  *small_max = small ? std::min(*wave_max, TRI_SMALL) : 0;
}

void tri_enqueue(const Prep& P, Scal* scal, const Tuning& tu, uint32_t flags, uint32_t cache_rows,
                 const TriWork& w, hipStream_t s) {
  const int64_t n = P.n;
  if (n == 0 || P.m == 0) return;
  if (!full_rows(P)) {  // one of several plans on these counters
    fill_u32(&scal->work[0], 0, 8, s);
    fill_u32(&scal->small.kmax, 0, 1, s);
  }
  int small_max, wave_max;
  tri_bounds(P, tu, flags, cache_rows, &small_max, &wave_max);
  k_tri_keys<<<(unsigned)ceil_div(n, 256), 256, 0, s>>>(P.dplus, n, P.own_lo, P.hi(), small_max,
                                                        wave_max, w.key, scal);
  radix_pass(w.key, nullptr, n, 0, 4, nullptr, w.order, w.rtmp, scal->small.tri_start, s);
  if (w.hoff) {
    int32_t* hsz = reinterpret_cast<int32_t*>(w.key);  // the keys are in order[] now
    k_hub_size<<<(unsigned)ceil_div(n, 256), 256, 0, s>>>(P.dplus, n, tu.hub_min, hsz, w.hub_list,
                                                          scal);
    scan_i32(hsz, n, w.hoff64, w.hst, s);
  }
}

Launch tri_plan(const Prep& P, Scal* scal, const Tuning& tu, uint32_t flags, uint32_t cache_rows,
                const TriWork& w, int num_cu, const std::function<char*(size_t)>& big_scratch,
                KTimer* kt, const SmallInfo& si, TriCredits* credits) {
  const int64_t n = P.n;
  if (n == 0 || P.m == 0) return [](hipStream_t) {};
  int32_t* order = w.order;
  const int64_t* start = scal->small.tri_start;
  int32_t* hoff = w.hoff;
  int32_t* hub_list = w.hub_list;
  int64_t* hoff64 = w.hoff64;
  int2* list = reinterpret_cast<int2*>(hoff64);  // takes its place once hoff is made of it
  int32_t* hsz = reinterpret_cast<int32_t*>(w.key);
  const bool hubs = hoff != nullptr;
  // largest out-degree of the global bucket decides its scratch size
  const unsigned int kmax_g = si.kmax;
  const int64_t* hstart = si.tri_start;
  const int64_t hub_slots = si.hub_slots;
  // scratch: hub tables, then the dense-owner bitmaps
  size_t hub_bytes = 0, dense_bytes = 0, dense_bits = 0, dense_blocks = 0;
  const bool use_hubs = hubs && hub_slots > 0 && hub_slots < (int64_t(1) << 31);
  if (use_hubs) hub_bytes = ((size_t)hub_slots * 8 + 255) & ~size_t(255);
  if (kmax_g > 0) {
    size_t K = kmax_g, WK = (K + 63) / 64;
    size_t per_block = K * WK * 8 + (7 * K + 2) * 4;
    int64_t owners = hstart[TK_GLOBAL + 1] - hstart[TK_GLOBAL];
    int64_t blocks = (int64_t)((size_t(1) << 30) / per_block);
    if (blocks > 64) blocks = 64;
    if (blocks > owners) blocks = owners;
    if (blocks < 1) blocks = 1;
    dense_blocks = (size_t)blocks;
    dense_bits = ((size_t)blocks * K * WK * 8 + 255) & ~size_t(255);
    dense_bytes = dense_bits + (size_t)blocks * (7 * K + 2) * 4;
  }
  char* scratch = nullptr;
  if (hub_bytes + dense_bytes > 0) {
    scratch = big_scratch(hub_bytes + dense_bytes);
    if (!scratch) throw Fail(M4_ENOMEM, "scratch for hub tables and dense out-lists does not fit");
  }

  TriArgs A{};
  A.order = order;
  A.start = start;
  A.nptr = P.nptr;
  A.optr = P.optr;
  A.ncol = P.ncol;
  A.dlo = P.dlo;
  A.dplus = P.dplus;
  A.t = P.t;
  A.scal = scal;
  A.err = &scal->err;
  A.flags = flags;
  A.cache_rows = cache_rows;
  A.list = list;
  if (use_hubs) {
    A.hoff = hoff;
    A.htab = reinterpret_cast<unsigned long long*>(scratch);
    A.hub_min = tu.hub_min;
    // a probe reads one line of a table: from the Infinity Cache while the
    // tables fit there, else from HBM, where it weighs more against a scan's
    // sequential reads
    A.probe_w = hub_bytes > kInfinityCacheBytes ? tu.probe_w_far : tu.probe_w;
  }
  std::array<int64_t, 17> hst;
  for (int i = 0; i < 17; i++) hst[i] = hstart[i];
  // the owners of one bucket in LDS: cred adds per-vertex credits
  auto run_lds = [=](TriArgs A, auto kmax_tag, auto nt_tag, auto cred_tag, int bucket,
                     int blocks_per_cu, int most, hipStream_t ls) {
    constexpr int KM = decltype(kmax_tag)::value;
    constexpr int NT = decltype(nt_tag)::value;
    const int64_t cnt = hst[bucket + 1] - hst[bucket];
    if (cnt == 0) return;
    const int64_t blocks = std::min<int64_t>((int64_t)num_cu * blocks_per_cu, cnt);
    A.bucket = bucket;
    A.work = &scal->work[bucket];
    // the work counter serves about 70 M atomics a second, so small owners
    // come several at once where there are many of them, and dealt in turn
    // where there are not (110000 owners of out-degree up to 64: 1.4 ms by
    // single grabs, 0.3 dealt; social 2^20 1.59 ms and 0.90)
    A.grab = (int)std::max<int64_t>(1, std::min<int64_t>(most, cnt / (blocks * 8)));
    if (cnt < blocks * most / 2) A.grab = 0;
    k_tri_lds<KM, NT, decltype(cred_tag)::value><<<(unsigned)blocks, NT, 0, ls>>>(A);
  };
  auto run_small = [=](TriArgs A, auto cred_tag, hipStream_t ls) {
    const int64_t cnt = hst[TK_SMALL + 1] - hst[TK_SMALL];
    if (cnt == 0) return;
    A.bucket = TK_SMALL;
    const int64_t blocks = std::min<int64_t>((int64_t)num_cu * 8, ceil_div(cnt, 256 / TRI_SMALL));
    k_tri_small<decltype(cred_tag)::value><<<(unsigned)blocks, 256, 0, ls>>>(A);
  };
  using std::integral_constant;
  using std::false_type;
  using std::true_type;
  if (credits) {
    credits->kmax = kmax_g > 0 ? (int)kmax_g : (hst[TK_1024 + 1] > hst[TK_1024] ? TRI_LDS_MAX : 0);
    credits->launch = [=](hipStream_t ls, unsigned long long* n12, unsigned long long* n14) {
      TriArgs B = A;
      B.n12 = n12;
      B.n14 = n14;
      fill_u32(&scal->work[0], 0, 8, ls);
      run_lds(B, integral_constant<int, 512>{}, integral_constant<int, 512>{}, true_type{}, TK_512,
              2, 1, ls);
      run_lds(B, integral_constant<int, 256>{}, integral_constant<int, 256>{}, true_type{}, TK_256,
              6, 1, ls);
      run_lds(B, integral_constant<int, 128>{}, integral_constant<int, 128>{}, true_type{}, TK_128,
              16, 8, ls);
      run_lds(B, integral_constant<int, 64>{}, integral_constant<int, 64>{}, true_type{}, TK_WAVE,
              32, 64, ls);
      run_small(B, true_type{}, ls);
    };
  }
  const bool planned = full_rows(P) && n <= SMALL_N;  // offsets and records are there
  // everything below runs on the launch stream, after the plan above
  return [=](hipStream_t ls) mutable {
    if (kt) kt->begin(M4_K_TRI_HUBS, ls);
    if (use_hubs && !planned)
      k_hub_off<<<(unsigned)ceil_div(n, 256), 256, 0, ls>>>(hsz, hoff64, n, hoff);
    if (list && !planned)
      k_tri_list<<<(unsigned)ceil_div(n + 1, 256), 256, 0, ls>>>(P.nptr, P.dlo, P.optr, n, list);
    if (use_hubs) {
      unsigned long long* htab = reinterpret_cast<unsigned long long*>(scratch);
      fill_u32(htab, 0xffffffffu, (size_t)hub_slots * 2, ls);
      k_hub_insert<<<(unsigned)(num_cu * 8), 256, 0, ls>>>(P.dplus, P.nptr, P.dlo, P.ncol, hoff,
                                                            hub_list, &scal->nhub, htab,
                                                            &scal->err);
    }
    if (kt) kt->end(M4_K_TRI_HUBS, ls);
    // heaviest buckets first so that their tails overlap the light ones
    if (kmax_g > 0) {
      const size_t K = kmax_g;
      TriArgs B = A;
      B.bucket = TK_GLOBAL;
      B.slot = M4_K_TRI_GLOBAL;
      B.grab = 1;
      B.work = &scal->work[TK_GLOBAL];
      B.kmax = (int)K;
      B.gbits = reinterpret_cast<uint64_t*>(scratch + hub_bytes);
      B.garr = reinterpret_cast<int32_t*>(scratch + hub_bytes + dense_bits);
      if (kt) kt->begin(M4_K_TRI_GLOBAL, ls);
      k_tri_global<256><<<(unsigned)dense_blocks, 256, 0, ls>>>(B);
      if (kt) kt->end(M4_K_TRI_GLOBAL, ls);
    }
    auto timed = [&](auto kmax_tag, auto nt_tag, int bucket, int slot, int blocks_per_cu, int most) {
      const bool any = hst[bucket + 1] > hst[bucket];
      A.slot = slot;
      if (kt && any) kt->begin(slot, ls);
      run_lds(A, kmax_tag, nt_tag, false_type{}, bucket, blocks_per_cu, most, ls);
      if (kt && any) kt->end(slot, ls);
    };
    if (hst[TK_1024 + 1] > hst[TK_1024]) {
      TriArgs B = A;
      B.bucket = TK_1024;
      B.slot = M4_K_TRI_1024;
      B.work = &scal->work[TK_1024];
      if (kt) kt->begin(M4_K_TRI_1024, ls);
      k_tri_large<1024, 256><<<(unsigned)std::min<int64_t>(num_cu, hst[TK_1024 + 1] - hst[TK_1024]),
                               256, 0, ls>>>(B);
      if (kt) kt->end(M4_K_TRI_1024, ls);
    }
    timed(integral_constant<int, 512>{}, integral_constant<int, 512>{}, TK_512, M4_K_TRI_512, 2, 1);
    timed(integral_constant<int, 256>{}, integral_constant<int, 256>{}, TK_256, M4_K_TRI_256, 8, 2);
    timed(integral_constant<int, 128>{}, integral_constant<int, 128>{}, TK_128, M4_K_TRI_128, 16, 16);
    // one slot for the owners of one wavefront and of a quarter of one
    const bool any = hst[TK_WAVE + 1] > hst[TK_WAVE] || hst[TK_SMALL + 1] > hst[TK_SMALL];
    A.slot = M4_K_TRI_WAVE;
    if (kt && any) kt->begin(M4_K_TRI_WAVE, ls);
    run_lds(A, integral_constant<int, 64>{}, integral_constant<int, 64>{}, false_type{}, TK_WAVE, 32,
            64, ls);
    run_small(A, false_type{}, ls);
    if (kt && any) kt->end(M4_K_TRI_WAVE, ls);
  };
}

}  // namespace m4
