// m4_c4.hip -- non-induced 4-cycle anchor (C4_ni).
//
// A 4-cycle is counted once, at its highest-ranked vertex u with opposite
// corner w: for every w < u let c_u[w] be the number of common neighbours v
// of u and w with v < u; each pair of them closes one cycle u-v-w-v', so
//   C4_ni = sum_u sum_w C(c_u[w], 2)
// (degree-ordered wedges, Chiba and Nishizeki 1985).  This is the cycle term
// of the paper's edge closure (Section III-F, adjacent pairs of A_e x B_e),
// reached through wedges instead of edge anchors.  The wedge endpoints of u
// are the prefixes below u of the sorted rows of its lower neighbours.  The
// sum is accumulated incrementally: every increment of c_u[w] adds the old
// value, so no second pass over the counters is needed.
//
// Vertices of degree <= 1 have rank < r1 and never contribute (c <= 1), so
// endpoints below r1 are skipped.  Owners are split by the wedge bound
// W_u = sum_{v in L(u)} (d(v) - 1):
//   tiny bucket   -- W_u <= 256: one wavefront, a table in LDS;
//   light, medium and large filter buckets -- one workgroup of 64, 256 or
//                    1024 threads: LDS bitmaps tell the endpoints met once
//                    from the others, which a table then counts;
//   window bucket -- large W_u dense over the ranks: one 1024-thread
//                    workgroup, dense counters in LDS over windows of
//                    128 KiB; a counter is 4 bits wide for endpoints of
//                    degree <= 15, 8 bits for degree <= 255 and 32 bits
//                    beyond (c_u[w] never exceeds d(w)), so a window spans up
//                    to 262144 ranks; every lower neighbour keeps a cursor
//                    into its sorted row so each window reads exactly its own
//                    endpoints.
// A filter costs per wedge; a window costs per rank of the owner's range, so
// owners whose endpoints are sparse over many windows belong in a filter.
#include <limits.h>
#include <string.h>

#include <algorithm>
#include <array>
#include <type_traits>

#include "m4_plan_dev.h"
#include "m4_walk_dev.h"

namespace m4 {

namespace {

struct C4Args {
  const int32_t* order;
  const int64_t* start;
  const int64_t* nptr;
  const int32_t* ncol;
  const int32_t* dr;
  const int32_t* dlo;
  const int2* wub;         // {wedge bound, lower neighbours of degree above 1}
  const int32_t* row_len;  // stored prefix of every row (null: full rows)
  int64_t r1;
  int bucket;
  int slot;
  unsigned int* work;
  Scal* scal;
  uint32_t flags;
  const int64_t* seg_off;  // window owners: first descriptor of each owner
  int4* desc;              // ... per-segment cursor descriptors
  const int32_t* seg_cnt;  // ... non-empty segments of each owner
  // large filtered owners: parts {owner, first rank, end rank, endpoints
  // expected}, the rank ranges that are counted apart (null: whole owners)
  const int4* parts;
  int64_t npart;           // parts of this bucket
  const int4* vmeta;       // per full row: offset, degree, lower neighbours, entries below r1
  unsigned long long* n8;  // per-vertex 4-cycle credits (orbit counts), or null
  int yb;                  // filtered owners: bits of a permuted rank
  int grab;                // tiny owners: owners of a run
  int class_cap;           // candidates a class of a filtered owner is planned for (0, or more
                           // than its table holds: 3/4 of that)
  // counter zones of the window owners (ranks >= r1): 4-bit counters for
  // ranks [r1, z1) (degree <= 15), 8-bit for [z1, z2) (degree <= 255), 32-bit
  // from z2 on; aw and bw are the words of the first two zones
  int32_t z1, z2, aw, bw, zr1;  // zr1: r1 as a 32-bit rank
};

constexpr uint32_t C4_MAX_CLASSES = 1u << 16;
constexpr uint32_t C4_KEY_MUL = 0x9E3779B1u, C4_KEY_INV = 0x0E8B2F51u;  // MUL x INV = 1 mod 2^32
// Direct counters: small graphs, and parts of large filtered owners over at
// most C4_DIRECT_SPAN ranks.
constexpr int32_t C4_DIRECT_SPAN = 262144;
// endpoints of one part of a large filtered owner; most parts
constexpr int64_t C4_BIN_RANGE = 131072;
constexpr int C4_MAX_PARTS = 4096;

// Wedge bound of every owner and its lower neighbours of degree above 1, the
// last of its lower entries (an entry of degree 1 is below r1 and holds no
// endpoint): the kernels read only those.  The bound stays below 2^31, since
// every CSR entry is an endpoint of an owner once at most.  A hub of 10^6 leaves
// with 180 wedges took its one wavefront 52 ms with the leaves.
// G lanes cooperate on one row, 4 loads in flight.
template <int G>
__global__ __launch_bounds__(256) void k_c4_plan(const int64_t* __restrict__ nptr,
                                                 const int32_t* __restrict__ ncol,
                                                 const int32_t* __restrict__ dr,
                                                 const int32_t* __restrict__ dlo, int64_t r_lo,
                                                 int64_t r_hi, int64_t r1, C4Plan pl,
                                                 int2* __restrict__ wub,
                                                 uint32_t* __restrict__ key, int64_t own_lo,
                                                 int64_t own_hi) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t u = r_lo + t / G;
  int j = (int)(t % G);
  bool ok = u < r_hi;
  if (ok && (u < own_lo || u >= own_hi)) {
    if (j == 0) key[u] = CB_NONE;
    ok = false;
  }
  int nl = ok ? dlo[u] : 0;
  int64_t b = ok ? nptr[u] : 0;
  int64_t s = 0;
  int nw = 0;
  int i = j;
  for (; i + 3 * G < nl; i += 4 * G) {
    int32_t v0 = ncol[b + i], v1 = ncol[b + i + G], v2 = ncol[b + i + 2 * G], v3 = ncol[b + i + 3 * G];
    s += (int64_t)dr[v0] + dr[v1] + dr[v2] + dr[v3] - 4;
    nw += (v0 >= r1) + (v1 >= r1) + (v2 >= r1) + (v3 >= r1);
  }
  for (; i < nl; i += G) {
    const int32_t v = ncol[b + i];
    s += dr[v] - 1;
    nw += v >= r1;
  }
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) {
    s += __shfl_xor(s, o, WAVE);
    nw += __shfl_xor(nw, o, WAVE);
  }
  if (ok && j == 0) {
    wub[u] = make_int2((int)s, nw);
    uint32_t k = CB_NONE;
    if (u >= r1 && nl >= 2 && s > 0) k = c4_bucket(pl, s, u, nw);
    key[u] = k;
  }
}

// rows too long for one wavefront: one 1024-thread workgroup per row
__global__ __launch_bounds__(1024) void k_c4_plan_big(const int64_t* __restrict__ nptr,
                                                      const int32_t* __restrict__ ncol,
                                                      const int32_t* __restrict__ dr,
                                                      const int32_t* __restrict__ dlo, int64_t r_lo,
                                                      int64_t r1, C4Plan pl,
                                                      int2* __restrict__ wub,
                                                      uint32_t* __restrict__ key, int64_t own_lo,
                                                      int64_t own_hi) {
  int64_t u = r_lo + blockIdx.x;
  if (u < own_lo || u >= own_hi) {
    if (threadIdx.x == 0) key[u] = CB_NONE;
    return;
  }
  int nl = dlo[u];
  int64_t b = nptr[u];
  int64_t s = 0;
  // both sums stay below 2^31: one scan of the pair
  for (int i = threadIdx.x; i < nl; i += 1024) {
    const int32_t v = ncol[b + i];
    s += dr[v] - 1 + ((int64_t)(v >= r1) << 32);
  }
  int64_t both;
  block_excl_scan64<1024>(s, &both);
  if (threadIdx.x == 0) {
    const int64_t tot = (uint32_t)both;
    const int nw = (int)(both >> 32);
    wub[u] = make_int2((int)tot, nw);
    uint32_t k = CB_NONE;
    if (u >= r1 && nl >= 2 && tot > 0) k = c4_bucket(pl, tot, u, nw);
    key[u] = k;
  }
}

__device__ __forceinline__ int64_t readlane64(int64_t v, int l) {
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)v, l);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// ---------------------------------------------------- segment walks
// The lower neighbours of an owner, taken from the highest rank down (the
// longest rows first, so that the short ones fill the walk's tail), as
// segments [first entry >= r1, row end) of the rank-space column array.
// Segments are not cut at the owner: a walk stops by value.

// Segments [s0, s0 + cnt) of owner row [base, base + nl) into LDS (and their
// vertices, where VERT), from their first entry >= lo on, an empty one after
// them; with pc > 1 (full rows) each is cut below hi and into pc pieces of about
// equal length, which count as segments.  Called by every thread of the
// workgroup.
template <int NT, bool VERT>
__device__ __forceinline__ void load_segs(const C4Args& A, int64_t base, int nl, int s0, int cnt,
                                          int32_t lo, int2* sg, int32_t* sv, int pc = 1,
                                          int32_t hi = 0) {
  if (threadIdx.x == 0) sg[cnt] = make_int2(0, 0);
  if (__builtin_expect(pc > 1, 0)) {
    for (int j = threadIdx.x; j < cnt; j += NT) {
      const int s = s0 + j, k = s % pc;
      const int32_t v = A.ncol[base + nl - 1 - s / pc];
      const int64_t rs = A.nptr[v], re = rs + A.dr[v];
      const int64_t c = lower_index(A.ncol, rs, re, lo);
      const int64_t len = lower_index(A.ncol, c, re, hi) - c;
      sg[j] = make_int2((int)(c + len * k / pc), (int)(c + len * (k + 1) / pc));
      if (VERT) sv[j] = v;
    }
    return;
  }
  for (int j = threadIdx.x; j < cnt; j += NT) {
    const int32_t v = A.ncol[base + nl - 1 - s0 - j];
    if (A.vmeta) {
      const int4 m = A.vmeta[v];  // row offset, degree, lower neighbours, entries below r1
      const int64_t c = m.x + m.w, e = m.x + m.y;
      sg[j] = make_int2((int)(lo > A.zr1 ? lower_index(A.ncol, c, e, lo) : c), (int)e);
    } else {
      // a partition stores row prefixes: one at most as long as the owner needs
      const int64_t rs = A.nptr[v];
      const int64_t e = rs + (A.row_len ? A.row_len[v] : A.dr[v]);
      sg[j] = make_int2((int)lower_index(A.ncol, rs, e, lo), (int)e);
    }
    if (VERT) sv[j] = v;
  }
}

__device__ __forceinline__ unsigned long long pairs_of(unsigned long long c) {
  return c * (c - 1) / 2;
}

template <int GL>
__device__ __forceinline__ unsigned long long lane_group_sum(unsigned long long v) {
#pragma unroll
  for (int o = GL / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}

// --------------------------------------------------------- tiny bucket
// One wavefront per owner with at most C4_TINY_MAX wedges: all endpoints in
// an open-addressing table in LDS, sized to twice the bound.  CRED adds the
// per-vertex credits to n8: C(c, 2) to the endpoint and the owner, the other
// wedges of its endpoint to each middle vertex.
template <bool CRED>
__global__ __launch_bounds__(WAVE) void k_c4_tiny(C4Args A) {
  constexpr int SLOTS = 2 * C4_TINY_MAX, SEGS = WAVE;
  __shared__ int32_t hkey[SLOTS];
  __shared__ uint32_t hcnt[SLOTS];
  __shared__ int2 sg[SEGS + 1];
  __shared__ int32_t sv[CRED ? SEGS : 1];
  __shared__ int s_next;
  const int lane = threadIdx.x;
  const int64_t b0 = A.start[A.bucket], cnt = A.start[A.bucket + 1] - b0;
  u128_t acc = 0;
  unsigned long long wedges = 0, owners = 0, segs = 0;
  for (int i = lane; i < SLOTS; i += WAVE) {
    hkey[i] = -1;
    hcnt[i] = 0;
  }
  // the owners cost about the same: runs of A.grab owners, dealt to the
  // wavefronts in turn
  for (int64_t first = (int64_t)blockIdx.x * A.grab; first < cnt;
       first += (int64_t)gridDim.x * A.grab) {
    // the owners of a run, one per lane
    const int64_t mine = first + lane;
    const bool have = lane < A.grab && mine < cnt;
    const int32_t mu = have ? A.order[b0 + mine] : 0;
    const int2 mw = have ? A.wub[mu] : make_int2(0, 0);
    const int32_t mwb = mw.x, mnl = mw.y;
    const int64_t mbase = have ? A.nptr[mu] + A.dlo[mu] - mnl : 0;
    const int nown = (int)std::min<int64_t>(A.grab, cnt - first);
    for (int o = 0; o < nown; o++) {
      const int32_t u = __builtin_amdgcn_readlane(mu, o);
      const int nl = __builtin_amdgcn_readlane(mnl, o);
      const int32_t wb = __builtin_amdgcn_readlane(mwb, o);
      const int64_t base = readlane64(mbase, o);
      int S = 64;
      while (S < 2 * wb) S <<= 1;
      const uint32_t mask = (uint32_t)S - 1;
      const int shift = 32 - (__ffs(S) - 1);
      owners++;
      segs += (unsigned long long)nl;
      // at most wb <= S / 2 distinct keys: a probe meets x or a free slot
      // within S steps
      auto insert = [&](int32_t x) {
        uint32_t h = ((uint32_t)x * 0x9E3779B1u) >> shift;
        for (int probes = 0; probes < S; probes++) {
          const int32_t k = hkey[h];
          if (k == x) return atomicAdd(&hcnt[h], 1u);
          if (k == -1) {
            const int32_t prev = atomicCAS(&hkey[h], -1, x);
            if (prev == -1 || prev == x) return atomicAdd(&hcnt[h], 1u);
          }
          h = (h + 1) & mask;
        }
        atomicOr(&A.scal->err, ERR_PROBE);
        return 0u;
      };
      for (int s0 = 0; s0 < nl; s0 += SEGS) {
        const int nc = nl - s0 < SEGS ? nl - s0 : SEGS;
        load_segs<WAVE, CRED>(A, base, nl, s0, nc, A.zr1, sg, sv);
        if (lane == 0) s_next = 0;
        wave_sync();
        unsigned part = 0;  // at most the pairs of C4_TINY_MAX endpoints
        seg_walk<8>(A.ncol, u, nc, &s_next, [&](int i) { return sg[i]; },
                    [&](const int32_t(&x)[4], int, int) {
#pragma unroll
                      for (int k = 0; k < 4; k++)
                        if (x[k] < u) {
                          wedges++;
                          part += insert(x[k]);
                        }
                    },
                    [](int, bool) {});
        acc += part;
        wave_sync();
      }
      if (CRED) {
        for (int s0 = 0; s0 < nl; s0 += SEGS) {
          const int nc = nl - s0 < SEGS ? nl - s0 : SEGS;
          if (nl > SEGS) load_segs<WAVE, CRED>(A, base, nl, s0, nc, A.zr1, sg, sv);
          if (lane == 0) s_next = 0;
          wave_sync();
          unsigned long long cr = 0;
          seg_walk<8>(A.ncol, u, nc, &s_next, [&](int i) { return sg[i]; },
                      [&](const int32_t(&x)[4], int, int) {
#pragma unroll
                        for (int k = 0; k < 4; k++)
                          if (x[k] < u) {
                            uint32_t h = ((uint32_t)x[k] * 0x9E3779B1u) >> shift;
                            for (int pr = 0; hkey[h] != x[k] && pr < S; pr++) h = (h + 1) & mask;
                            cr += hcnt[h] - 1;
                          }
                      },
                      [&](int i, bool last) {
                        if (!__ballot(last)) return;
                        const unsigned long long t = lane_group_sum<8>(cr);
                        if (last) {
                          if ((lane & 7) == 0 && t) atomicAdd(&A.n8[sv[i]], t);
                          cr = 0;
                        }
                      });
          wave_sync();
        }
        unsigned long long own = 0;
        for (int i = lane; i < S; i += WAVE) {
          const unsigned long long c = hcnt[i];
          if (c >= 2) {
            own += pairs_of(c);
            atomicAdd(&A.n8[hkey[i]], pairs_of(c));
          }
        }
        own = lane_group_sum<WAVE>(own);
        if (lane == 0 && own) atomicAdd(&A.n8[u], own);
      }
      for (int i = lane; i < S; i += WAVE) {
        hkey[i] = -1;
        hcnt[i] = 0;
      }
      wave_sync();
    }
  }
  block_add_acc<WAVE>(A.scal, ACC_C4, acc);
  if (A.flags & M4_STATS) {
    block_add_u64<WAVE>(&A.scal->stat[ST_WEDGES], wedges);
    block_add_u64<WAVE>(&A.scal->kstat[A.slot][0], wedges);
    block_add_u64<WAVE>(&A.scal->kstat[A.slot][1], lane == 0 ? owners : 0);
    block_add_u64<WAVE>(&A.scal->kstat[A.slot][2], lane == 0 ? segs : 0);
    block_add_u64<WAVE>(&A.scal->kstat[A.slot][3], wedges);
  }
}

// ------------------------------------------------------- direct counters
// The endpoints of owner u in ranks [lo, end) counted with one 32-bit LDS
// counter per rank, over windows of WORDS ranks: one walk counts (the old
// values are the sum), CRED takes a second walk for the middle vertices and a
// sweep of the counters for endpoints and owner.  Where a window holds many
// endpoints per rank this beats a filter, which would count nearly all of
// them in its table.  Called by every thread of the workgroup; the counters
// need not be clear.
template <int NT, int WORDS, int SEGS, bool CRED>
__device__ __forceinline__ void count_direct(const C4Args& A, uint4* cnt4, int2* sg, int32_t* sv,
                                             int* next, int64_t base, int nl, int32_t lo,
                                             int32_t end, u128_t& acc, unsigned long long& wedges,
                                             unsigned long long& own) {
  uint32_t* cnt = reinterpret_cast<uint32_t*>(cnt4);
  const int tid = threadIdx.x, lane = tid & (WAVE - 1);
  for (; lo < end; lo += WORDS) {
    const int32_t hi = end - lo < WORDS ? end : lo + WORDS;
    for (int i = tid; i < (hi - lo + 3) / 4; i += NT) cnt4[i] = make_uint4(0, 0, 0, 0);
    bool loaded = false;
    auto walk = [&](auto&& ent, auto&& fin) {
      for (int s0 = 0; s0 < nl; s0 += SEGS) {
        const int nc = nl - s0 < SEGS ? nl - s0 : SEGS;
        if (!loaded) load_segs<NT, CRED>(A, base, nl, s0, nc, lo, sg, sv);
        loaded = nl <= SEGS;
        if (tid == 0) *next = 0;
        __syncthreads();
        seg_walk<8>(A.ncol, hi, nc, next, [&](int i) { return sg[i]; }, ent, fin);
        __syncthreads();
      }
    };
    unsigned long long part = 0;
    walk(
        [&](const int32_t(&x)[4], int, int) {
          uint32_t old[4];
#pragma unroll
          for (int k = 0; k < 4; k++) {
            const bool in = x[k] < hi;
            old[k] = in ? atomicAdd(&cnt[x[k] - lo], 1u) : 0u;
            wedges += in;
          }
#pragma unroll
          for (int k = 0; k < 4; k++) part += old[k];
        },
        [](int, bool) {});
    acc += part;
    if (CRED) {
      unsigned long long cr = 0;
      walk(
          [&](const int32_t(&x)[4], int, int) {
#pragma unroll
            for (int k = 0; k < 4; k++)
              if (x[k] < hi) cr += cnt[x[k] - lo] - 1;
          },
          [&](int i, bool last) {
            if (!__ballot(last)) return;
            const unsigned long long t = lane_group_sum<8>(cr);
            if (last) {
              if ((lane & 7) == 0 && t) atomicAdd(&A.n8[sv[i]], t);
              cr = 0;
            }
          });
      for (int i = tid; i < hi - lo; i += NT) {
        const unsigned long long c = cnt[i];
        if (c >= 2) {
          own += pairs_of(c);
          atomicAdd(&A.n8[lo + i], pairs_of(c));
        }
      }
    }
    __syncthreads();
  }
}

// Graphs of at most SMALL_N vertices: every owner above the tiny bound,
// whatever its bucket (one window, no cursors, no bitmaps, one launch).
template <bool CRED>
__global__ __launch_bounds__(256) void k_c4_direct(C4Args A) {
  constexpr int NT = 256, SEGS = 256;
  __shared__ uint4 cnt4[SMALL_N / 4];
  __shared__ int2 sg[SEGS + 1];
  __shared__ int32_t sv[CRED ? SEGS : 1];
  __shared__ int s_next;
  const int tid = threadIdx.x, lane = tid & (WAVE - 1);
  const int64_t b0 = A.start[CB_HASH], items = A.start[CB_N] - b0;
  u128_t acc = 0;
  for (int64_t item = blockIdx.x; item < items; item += gridDim.x) {
    const int64_t at = b0 + items - 1 - item;  // heaviest owners (highest ranks) first
    const int32_t u = __builtin_amdgcn_readfirstlane(A.order[at]);
    const int nl = __builtin_amdgcn_readfirstlane(A.wub[u].y);
    unsigned long long own = 0, wedges = 0;
    count_direct<NT, SMALL_N, SEGS, CRED>(A, cnt4, sg, sv, &s_next, A.nptr[u] + A.dlo[u] - nl, nl,
                                          A.zr1, u, acc, wedges, own);
    if (CRED) {
      own = lane_group_sum<WAVE>(own);
      if (lane == 0 && own) atomicAdd(&A.n8[u], own);
    }
    if (A.flags & M4_STATS) {
      // the slot of the owner's bucket
      const int slot = at < A.start[CB_HASH + 1]  ? M4_K_C4_HASH
                       : at < A.start[CB_MED + 1] ? M4_K_C4_MED
                       : at < A.start[CB_WIN + 1] ? M4_K_C4_WINDOW
                                                  : M4_K_C4_BIN;
      const unsigned long long one = tid == 0 ? 1 : 0;
      block_add_u64<NT>(&A.scal->stat[ST_WEDGES], wedges);
      block_add_u64<NT>(&A.scal->kstat[slot][0], wedges);
      block_add_u64<NT>(&A.scal->kstat[slot][1], one);
      block_add_u64<NT>(&A.scal->kstat[slot][2], one * (unsigned long long)nl);
      block_add_u64<NT>(&A.scal->kstat[slot][3], one);
    }
  }
  block_add_acc<NT>(A.scal, ACC_C4, acc);
}

// ------------------------------------------------------- filter buckets
// Most wedge endpoints of a sparse owner are met once (88 % on the scale-24
// web graph) and close no 4-cycle, so they are told apart before anything is
// counted.  Per owner, one workgroup:
//   1. a walk over the endpoints sets one bit per endpoint in an LDS bitmap
//      (bit x mod 2^AB of rank x); an endpoint that finds its bit set also
//      sets bit x mod 2^BB of a second one;
//   2. a second walk counts exactly the endpoints whose bit is set in the
//      second bitmap (those met twice, and a few that share bits with others)
//      in a table laid over the first bitmap;
//   3. CRED: a third walk adds to each middle vertex the other wedges of its
//      endpoints, and a sweep of the table C(c, 2) to endpoints and owner.
// Table slots: a rank is held as y = x K mod 2^yb (K odd: a bijection), home
// slot = the high bits of y; a 32-bit slot keeps the rest of y, its distance
// from the home slot (6 bits) and the count above them, which stays below
// the owner's lower neighbours (the plan sends no owner whose number does
// not fit).  WIDE slots hold rank + 1 and a 32-bit count.
// An owner with more than C4_BIN_RANGE endpoints is counted in parts: rank
// ranges of about equal numbers of endpoints, each by any workgroup, so that
// no single owner keeps one CU busy after the others have ended.  A part with
// more candidates than the table holds is counted in P classes of a second
// hash, one walk each; a class that overflows the table is dropped, split in two
// and walked again, so every owner ends.
// Bound by vector issue (52 % of the CU's cycles) and, at 16 wavefronts a CU, by
// the latency of a walk's one load in flight.  Scale-24 web graph (268 M edges):
// the 395 K large owners (21.5 G endpoints, about 2.5 walks each) 83 ms, 209 ms
// when their endpoints were sorted into bins in device memory; the 698 K medium
// ones (1.76 G) 7.5 ms, 33 ms in 16384-slot tables with a search per endpoint;
// light and tiny ones 2.5 and 2.6 ms, 18 ms together.  While the lanes without an
// endpoint shared a word (91, 8.8 and 4.1 ms, a third of the large ones' LDS
// cycles more in conflicts): parts of 98 K / 131 K / 196 K endpoints 97 / 91 /
// 104 ms; direct counters for parts of up to 33 K / 131 K / 262 K / 524 K ranks
// 98 / 95 / 91 / 99 ms; 512-thread workgroups, two a CU with half the bitmap,
// 167 ms (at 103); whole owners instead of parts 103 ms, and the credits of the
// web 2^21 graph 51 ms instead of 20, of the social 2^18 graph 38 instead of 2.6
// (one hub kept one CU busy); with one global atomic per wedge into n counters
// per workgroup they took 336 and 19 ms.
template <int AB, bool WIDE>
struct FilterTable {
  using Slot = std::conditional_t<WIDE, unsigned long long, uint32_t>;
  static constexpr int HB = AB - 5 - (WIDE ? 1 : 0);  // home slot bits
  static constexpr int N = 1 << HB;
  static constexpr int PROBES = 1 << C4_DISP_BITS;
  Slot* t;
  uint32_t ymask, qmask;
  int qb, cs;  // bits of y below the home slot; first bit of the count
  __device__ __forceinline__ FilterTable(void* mem, int yb)
      : t(static_cast<Slot*>(mem)),
        ymask(yb >= 32 ? ~0u : (1u << yb) - 1u),
        qmask(WIDE ? 0u : (1u << (yb - HB)) - 1u),
        qb(yb - HB),
        cs(WIDE ? 0 : yb - HB + C4_DISP_BITS) {}
  // calls hit(slot pointer, its word) on the slot of x; false if none within
  // PROBES of the home slot.  INS claims an empty slot (count 1, old count 0).
  template <bool INS>
  __device__ __forceinline__ bool find(int32_t x, unsigned long long& got) {
    const uint32_t y = ((uint32_t)x * C4_KEY_MUL) & ymask;
    uint32_t h = y >> qb;
    const Slot one = WIDE ? Slot(1) : Slot(1) << cs;
    const Slot idm = WIDE ? ~Slot(0xffffffffu) : one - 1;
    Slot id = WIDE ? Slot((unsigned long long)(uint32_t)(x + 1) << 32) : Slot(y & qmask);
    for (int d = 0; d < PROBES; d++) {
      Slot w = t[h];
      if (INS && w == 0) {
        w = atomicCAS(&t[h], Slot(0), one | id);
        if (w == 0) {
          got = 0;
          return true;
        }
      }
      if ((w & idm) == id) {
        if (INS) w = atomicAdd(&t[h], one);
        got = count_of(w);
        return true;
      }
      h = (h + 1) & (N - 1);
      if (!WIDE) id += Slot(1) << qb;
    }
    return false;
  }
  __device__ __forceinline__ unsigned long long count_of(Slot w) const {
    return WIDE ? (unsigned long long)(uint32_t)w : (unsigned long long)(w >> cs);
  }
  // the rank kept in slot i with word w
  __device__ __forceinline__ uint32_t rank_of(int i, Slot w) const {
    if (WIDE) return (uint32_t)((unsigned long long)w >> 32) - 1u;
    const uint32_t home = ((uint32_t)i - ((uint32_t)(w >> qb) & (PROBES - 1u))) & (N - 1u);
    return (((home << qb) | ((uint32_t)w & qmask)) * C4_KEY_INV) & ymask;
  }
};

template <int NT, int GL, int AB, int BB, int SEGS, bool CRED, bool WIDE = false>
__global__ __launch_bounds__(NT) void k_c4_filter(C4Args A) {
  using Table = FilterTable<AB, WIDE>;
  constexpr int AW = 1 << (AB - 5), BW = 1 << (BB - 5);  // bitmap words
  // (a larger plan than the table would overflow and be walked for nothing)
  const unsigned long long CAP =
      A.class_cap > 0 && A.class_cap <= Table::N ? A.class_cap : Table::N / 4 * 3;
  __shared__ uint4 fa4[AW / 4];
  __shared__ uint4 fb4[BW / 4];
  __shared__ int2 sg[SEGS + 1];
  __shared__ int32_t wq[NT / WAVE][2 * WAVE];  // per wavefront: candidates to count
  __shared__ int32_t sv[CRED ? SEGS : 1];
  __shared__ int s_item, s_next, s_over;
  __shared__ unsigned s_dup, s_bits;
  uint32_t* fa = reinterpret_cast<uint32_t*>(fa4);
  uint32_t* fb = reinterpret_cast<uint32_t*>(fb4);
  const int tid = threadIdx.x, lane = tid & (WAVE - 1);
  const int64_t b0 = A.start[A.bucket];
  const int64_t cnt = A.parts ? A.npart : A.start[A.bucket + 1] - b0;
  Table tab(fa4, A.yb);
  u128_t acc = 0;
  unsigned long long wedges = 0, owners = 0, segs = 0, walks = 0;
  // the first owner of a workgroup is its own; large owners then come from
  // the work counter, asked one owner ahead; the many small ones are dealt
  // in turn, since one counter serves only about 70 M atomics a second
  constexpr bool DEAL = NT <= 256;
  for (int64_t item = blockIdx.x; item < cnt;) {
    unsigned ahead = 0;
    if (!DEAL && tid == 0) ahead = atomicAdd(A.work, 1u);
    const int64_t pos = cnt - 1 - item;  // heaviest owners (highest ranks) first
    int4 part;
    if (A.parts) part = A.parts[pos];
    else part.x = A.order[b0 + pos];
    const int32_t u = __builtin_amdgcn_readfirstlane(part.x);
    const int2 bound = A.wub[u];
    const int nl = __builtin_amdgcn_readfirstlane(bound.y);
    const int64_t base = A.nptr[u] + A.dlo[u] - nl;
    const int32_t lo = A.parts ? __builtin_amdgcn_readfirstlane(part.y) : A.zr1;
    const int32_t hi = A.parts ? __builtin_amdgcn_readfirstlane(part.z) : u;
    const unsigned long long wb =
        A.parts ? (unsigned long long)part.w : (unsigned long long)bound.x;
    if (lo == A.zr1) {  // an owner's first part
      owners++;
      segs += (unsigned long long)nl;
    }
    unsigned long long own = 0;
    if (NT == 1024 && hi - lo <= C4_DIRECT_SPAN) {
      // a dense part: the first bitmap's words as counters
      count_direct<NT, AW, SEGS, CRED>(A, fa4, sg, sv, &s_next, base, nl, lo, hi, acc, wedges, own);
      walks++;
    } else if (lo < hi) {
      // ---- 1. the bitmaps
      for (int i = tid; i < AW / 4; i += NT) fa4[i] = make_uint4(0, 0, 0, 0);
      for (int i = tid; i < BW / 4; i += NT) fb4[i] = make_uint4(0, 0, 0, 0);
      if (tid == 0) s_dup = s_bits = 0;
      // walks all segments, SEGS at a time; where they all fit they are
      // loaded once per range
      bool loaded = false;
      // A few long rows would leave most groups of lanes without a segment: two
      // rows of 140000 entries, orbits 82 ms whole and 12.7 in pieces (43 with a
      // thread per wedge)
      const int pc = NT == 1024 && nl <= 32 && wb >= 16384 ? SEGS / nl : 1, np = nl * pc;
      auto walk = [&](auto&& ent, auto&& fin) {
        for (int s0 = 0; s0 < np; s0 += SEGS) {
          const int nc = np - s0 < SEGS ? np - s0 : SEGS;
          if (!loaded) load_segs<NT, CRED>(A, base, nl, s0, nc, lo, sg, sv, pc, hi);
          loaded = np <= SEGS;
          if (tid == 0) s_next = 0;
          __syncthreads();
          seg_walk<GL>(A.ncol, hi, nc, &s_next, [&](int i) { return sg[i]; }, ent, fin);
          __syncthreads();
        }
        walks++;
      };
      // endpoints of one owner: each CSR entry once at most, so below 2^31
      unsigned dup = 0, valid = 0;
      walk(
          [&](const int32_t(&x)[4], int, int) {
            // lanes without an endpoint set nothing, each in a word of its own:
            // in one word they wait for each other, all but a few of a
            // wavefront's where segments are short (140000 segments of one
            // endpoint 19.4 -> 13 ms, web 2^24 206.5 -> 195.5 ms a call)
            uint32_t bit[4], old[4], at[4];
#pragma unroll
            for (int k = 0; k < 4; k++) {
              const bool in = x[k] < hi;
              bit[k] = in ? 1u << (x[k] & 31) : 0u;
              at[k] = in ? (uint32_t)x[k] >> 5 : (uint32_t)lane;
              valid += in;
              old[k] = atomicOr(&fa[at[k] & (AW - 1)], bit[k]);
            }
            // without a branch: a lane that finds its bit clear sets nothing
#pragma unroll
            for (int k = 0; k < 4; k++) {
              const uint32_t d = old[k] & bit[k];
              dup += d != 0;
              atomicOr(&fb[at[k] & (BW - 1)], d);
            }
          },
          [](int, bool) {});
      wedges += valid;
      dup = (unsigned)lane_group_sum<WAVE>(dup);
      if (lane == 0 && dup) atomicAdd(&s_dup, dup);
      __syncthreads();
      const unsigned long long nd = (unsigned)__builtin_amdgcn_readfirstlane((int)s_dup);
      // ---- 2. the candidates, in P classes
      // distinct candidates: an endpoint that found its bit set repeats a key
      // or shares the bit with another key, and of the endpoints met once some
      // have their bit of the smaller second bitmap set by others; never more
      // than the ranks of the range
      const unsigned long long est = std::min<unsigned long long>(
          nd + ((wb * nd) >> BB), (unsigned long long)(hi - lo));
      uint32_t P = (uint32_t)std::min<unsigned long long>((est + CAP - 1) / CAP, C4_MAX_CLASSES);
      if (nd == 0) P = 0;
      if (__builtin_expect(P > 4, 0)) {
        // Many classes: perhaps of few ranks, each met many times.  nb set bits
        // of the second bitmap's B = 2^BB, where they are few, stand for little
        // more than nb ranks (three times as many are allowed for), and a share
        // nb / B of the other endpoints has its bit set by them.  140000
        // endpoints of one rank took five classes: 13 -> 2.7 ms.  Asked of every
        // part, with a logarithm where bits are many, this took the web 2^24
        // graph from 195.5 to 199.5 ms.
        static_assert(BW == 4 * NT, "16 bytes of the second bitmap a thread");
        const uint4 v = fb4[tid];
        int set = __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
#pragma unroll
        for (int o = WAVE / 2; o > 0; o >>= 1) set += __shfl_xor(set, o, WAVE);
        if (lane == 0 && set) atomicAdd(&s_bits, (unsigned)set);
        __syncthreads();
        const uint32_t nb = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_bits);
        if (nb < (1u << (BB - 4)))
          P = std::min<uint32_t>(P, 1 + (3 * nb + (uint32_t)((wb * nb) >> BB)) / (uint32_t)CAP);
      }
      for (uint32_t c = 0; c < P;) {
        for (int i = tid; i < AW / 4; i += NT) fa4[i] = make_uint4(0, 0, 0, 0);
        if (tid == 0) s_over = 0;
        __syncthreads();
        auto candidate = [&](int32_t x) {
          const bool c1 = ((fb[((uint32_t)x >> 5) & (BW - 1)] >> (x & 31)) & 1) != 0 && x < hi;
          if (P == 1) return c1;
          return c1 && ((((uint32_t)x * 0x85EBCA6Bu) >> 16) * P) >> 16 == c;
        };
        // the candidates of a step are gathered in LDS and counted 64 at a
        // time, one per lane: a fraction of the entries are candidates, and
        // probing them in place would leave most lanes idle
        bool over = false;
        unsigned long long part = 0;
        int qn = 0;  // uniform in the wavefront
        int32_t* q = wq[tid / WAVE];
        auto count_top = [&](int m) {
          wave_sync();
          if (lane < m) {
            unsigned long long old = 0;
            if (tab.template find<true>(q[qn - m + lane], old)) part += old;
            else over = true;
          }
          qn -= m;
          wave_sync();
        };
        walk(
            [&](const int32_t(&x)[4], int, int) {
#pragma unroll
              for (int k = 0; k < 4; k++) {
                const bool is = candidate(x[k]);
                const uint64_t m = __ballot(is);
                if (is) q[qn + lanes_before(m)] = x[k];
                qn += __popcll(m);
                if (qn >= WAVE) count_top(WAVE);
              }
            },
            [](int, bool) {});
        if (qn > 0) count_top(qn);
        if (over) s_over = 1;
        __syncthreads();
        const int split = s_over;
        __syncthreads();
        if (split) {
          if (P > C4_MAX_CLASSES / 2) {  // not met by any owner the plan sends here
            if (tid == 0) atomicOr(&A.scal->err, ERR_RANGES);
            break;
          }
          P *= 2;  // class c is 2c and 2c + 1 of the finer split
          c *= 2;
          continue;
        }
        acc += part;
        if (CRED) {
          unsigned long long cr = 0;
          walk(
              [&](const int32_t(&x)[4], int, int) {
#pragma unroll
                for (int k = 0; k < 4; k++)
                  if (candidate(x[k])) {
                    unsigned long long n = 1;
                    (void)tab.template find<false>(x[k], n);
                    cr += n - 1;
                  }
              },
              [&](int i, bool last) {
                if (!__ballot(last)) return;
                const unsigned long long t = lane_group_sum<GL>(cr);
                if (last) {
                  if ((lane & (GL - 1)) == 0 && t) atomicAdd(&A.n8[sv[i]], t);
                  cr = 0;
                }
              });
          for (int i = tid; i < Table::N; i += NT) {
            const typename Table::Slot w = tab.t[i];
            const unsigned long long k = tab.count_of(w);
            if (k >= 2) {
              own += pairs_of(k);
              atomicAdd(&A.n8[tab.rank_of(i, w)], pairs_of(k));
            }
          }
          __syncthreads();
        }
        c++;
      }
    }
    if (CRED) {
      own = lane_group_sum<WAVE>(own);
      if (lane == 0 && own) atomicAdd(&A.n8[u], own);
    }
    if (DEAL) {
      item += gridDim.x;
    } else {
      __syncthreads();  // every thread has read the last s_item
      if (tid == 0) s_item = (int)(gridDim.x + ahead);
      __syncthreads();
      item = __builtin_amdgcn_readfirstlane(s_item);
    }
  }
  block_add_acc<NT>(A.scal, ACC_C4, acc);
  if (A.flags & M4_STATS) {
    const unsigned long long b0v = tid == 0 ? 1 : 0;
    block_add_u64<NT>(&A.scal->stat[ST_WEDGES], wedges);
    block_add_u64<NT>(&A.scal->kstat[A.slot][0], wedges);
    block_add_u64<NT>(&A.scal->kstat[A.slot][1], owners * b0v);
    block_add_u64<NT>(&A.scal->kstat[A.slot][2], segs * b0v);
    block_add_u64<NT>(&A.scal->kstat[A.slot][3], walks * b0v);
  }
}

// -------------------------------------------------------- window bucket
// Segment descriptors of the window owners: for lower neighbour v of owner u
// the cursor into row v (first entry >= r1), the row's end, and the values at
// the cursor and 7 entries after it.  Only non-empty segments are kept (a
// lower neighbour of degree 1, say, has none), packed from the owner's first
// slot; seg_cnt[h] is their number.  One block per owner.
__global__ __launch_bounds__(256) void k_c4_desc(const int32_t* __restrict__ order,
                                                 const int64_t* __restrict__ start,
                                                 const int64_t* __restrict__ seg_off,
                                                 const int64_t* __restrict__ nptr,
                                                 const int32_t* __restrict__ dlo,
                                                 const int32_t* __restrict__ ncol,
                                                 const int4* __restrict__ vmeta,
                                                 const int32_t* __restrict__ row_len, int64_t r1,
                                                 int4* __restrict__ desc,
                                                 int32_t* __restrict__ seg_cnt) {
  const int64_t h = blockIdx.x;
  const int32_t u = order[start[CB_WIN] + h];
  const int64_t so = seg_off[h], base = nptr[u];
  const int nl = dlo[u];
  int64_t kept = 0;
  for (int i0 = 0; i0 < nl; i0 += 256) {
    const int i = i0 + (int)threadIdx.x;
    int64_t c = 0, e = 0;
    if (i < nl) {
      const int32_t v = ncol[base + i];
      if (vmeta) {
        const int4 m = vmeta[v];
        e = m.x + m.y;
        c = m.x + m.w;
      } else {
        const int64_t rs = nptr[v];
        e = row_len ? rs + row_len[v] : nptr[v + 1];
        // first entry >= r1, searched in the stored prefix
        c = lower_index(ncol, rs, e, (int32_t)r1);
      }
    }
    int64_t ktot;
    const int64_t kx = block_excl_scan64<256>(c < e ? 1 : 0, &ktot);
    if (c < e)
      desc[so + kept + kx] =
          make_int4((int)c, (int)e, ncol[c], c + 7 < e ? ncol[c + 7] : INT_MAX);
    kept += ktot;
  }
  if (threadIdx.x == 0) seg_cnt[h] = (int32_t)kept;
}

// per full row: {row offset, degree, lower neighbours, entries below r1
// (degree <= 1) at its head}; row offsets fit 32 bits (CSR positions do)
__global__ void k_vmeta(const int64_t* __restrict__ nptr, const int32_t* __restrict__ ncol,
                        const int32_t* __restrict__ dr, const int32_t* __restrict__ dlo, int64_t n,
                        int64_t r1, int4* __restrict__ vmeta) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  const int64_t rs = nptr[v];
  const int32_t cut = (int32_t)(lower_index(ncol, rs, nptr[v + 1], (int32_t)r1) - rs);
  vmeta[v] = make_int4((int)rs, dr[v], dlo[v], cut);
}

// Lengths of the heavy owners' lists: segment descriptors of a window owner,
// parts of a large filtered one (the two are adjacent in the bucket order).
__global__ void k_c4_heavy_len(const int32_t* __restrict__ order, const int64_t* __restrict__ start,
                               const int32_t* __restrict__ dlo, const int2* __restrict__ wub,
                               int64_t H, int32_t* __restrict__ len) {
  const int64_t h = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (h >= H) return;
  const int32_t u = order[start[CB_WIN] + h];
  if (h < start[CB_WIN + 1] - start[CB_WIN]) {
    len[h] = dlo[u];
  } else {
    const int64_t k = (wub[u].x + C4_BIN_RANGE - 1) / C4_BIN_RANGE;
    len[h] = (int32_t)(k < C4_MAX_PARTS ? k : C4_MAX_PARTS);
  }
}

// The parts of the large filtered owners: rank ranges of about equal numbers
// of endpoints (an endpoint's chance to be rank x is about proportional to the
// degree of x, and the row offsets are the degrees' prefix sums).  One thread
// per part; off holds the first part of each owner.
__global__ void k_c4_parts(const int32_t* __restrict__ owner, const int2* __restrict__ wub,
                           const int64_t* __restrict__ nptr, const int64_t* __restrict__ off,
                           int64_t H, int64_t total, int64_t r1, int4* __restrict__ parts) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int64_t h = lower_index(off, (int64_t)0, H, i + 1) - 1;  // the owner whose parts hold i
  const int32_t u = owner[h];
  const int64_t p = i - off[h], k = off[h + 1] - off[h];
  const int64_t d0 = nptr[r1], d1 = nptr[u];
  auto cut = [&](int64_t q) -> int32_t {
    if (q <= 0) return (int32_t)r1;
    if (q >= k) return u;
    return (int32_t)lower_index(nptr, r1, (int64_t)u,
                                d0 + (int64_t)((double)(d1 - d0) * (double)q / (double)k));
  };
  const int64_t w = (wub[u].x + k - 1) / k;
  parts[i] = make_int4(u, cut(p), cut(p + 1), (int)(w < INT_MAX ? w : INT_MAX));
}

constexpr int W_NT = 1024, W_GL = 8, W_NG = W_NT / W_GL, W_SHORT = 8;
constexpr int W_LD = 2;  // 16-byte loads per lane and step of a long visit
constexpr int W_BATCH = 2048;  // segments per pass (bounds the long-visit queue)
constexpr int W_RPT = W_BATCH / W_NT;  // segments per thread and pass

// Counter of rank x (x >= r1) in the zoned layout: a 4-bit counter while the
// degree of x is <= 15, 8-bit while <= 255, else 32-bit.  c_u[x] counts
// common neighbours of u and x, so it never exceeds the degree of x and no
// counter overflows into its neighbour.
__device__ __forceinline__ void zone_slot(const C4Args& A, int32_t x, int32_t& word, int& shift) {
  if (x < A.z1) {
    const int32_t k = x - A.zr1;
    word = k >> 3;
    shift = (k & 7) * 4;
  } else if (x < A.z2) {
    const int32_t k = x - A.z1;
    word = A.aw + (k >> 2);
    shift = (k & 3) * 8;
  } else {
    word = A.aw + A.bw + (x - A.z2);
    shift = 0;
  }
}

// first rank whose counter lies in word w
__device__ __forceinline__ int32_t zone_rank(const C4Args& A, int32_t w) {
  if (w < A.aw) return A.zr1 + 8 * w;
  if (w < A.aw + A.bw) return A.z1 + 4 * (w - A.aw);
  return A.z2 + (w - A.aw - A.bw);
}

// words holding the counters of ranks [r1, u)
__device__ __forceinline__ int32_t zone_words(const C4Args& A, int32_t u) {
  if (u <= A.zr1) return 0;
  if (u <= A.z1) return (u - A.zr1 + 7) >> 3;
  if (u <= A.z2) return A.aw + ((u - A.z1 + 3) >> 2);
  return A.aw + A.bw + (u - A.z2);
}

// one wedge endpoint x of the window starting at word wlo: returns the old
// count c (every increment of c_u[x] from c to c + 1 adds c to the sum of
// C(c_u[x], 2))
__device__ __forceinline__ uint32_t window_inc(const C4Args& A, uint32_t* cnt, int32_t wlo,
                                               int32_t x) {
  int32_t word;
  int shift;
  zone_slot(A, x, word, shift);
  const uint32_t mask = x < A.z1 ? 0xfu : (x < A.z2 ? 0xffu : 0xffffffffu);
  const uint32_t old = atomicAdd(&cnt[word - wlo], 1u << shift);
  return (old >> shift) & mask;
}

// The same increment for a window that lies inside one zone (KIND 0: 4-bit
// counters, 1: 8-bit, 2: 32-bit; 3: the window crosses a zone bound): with
// base the first rank of the window's first word, the counter word is
// (x - base) >> log2(counters per word), so the zone tests and the shifted
// zone offsets drop out of the per-endpoint work.
template <int KIND>
__device__ __forceinline__ uint32_t window_inc_k(const C4Args& A, uint32_t* cnt, int32_t wlo,
                                                 int32_t base, int32_t x) {
  if constexpr (KIND == 0) {
    const int32_t k = x - base;
    const int sh = (k & 7) << 2;
    return (atomicAdd(&cnt[k >> 3], 1u << sh) >> sh) & 0xfu;
  } else if constexpr (KIND == 1) {
    const int32_t k = x - base;
    const int sh = (k & 3) << 3;
    return (atomicAdd(&cnt[k >> 2], 1u << sh) >> sh) & 0xffu;
  } else if constexpr (KIND == 2) {
    return atomicAdd(&cnt[x - base], 1u);
  } else {
    return window_inc(A, cnt, wlo, x);
  }
}

// word holding the counter of rank x (x >= r1)
__device__ __forceinline__ int32_t zone_word(const C4Args& A, int32_t x) {
  int32_t word;
  int shift;
  zone_slot(A, x, word, shift);
  return word;
}

__device__ __forceinline__ int32_t row_at(const int32_t* ncol, int64_t i, int64_t e) {
  return i < e ? ncol[i] : INT_MAX;
}

__device__ __forceinline__ int32_t comp(const int4& v, int r) {
  return r == 0 ? v.x : (r == 1 ? v.y : (r == 2 ? v.z : v.w));
}

// A visit of at most 7 entries by one thread: entries c .. c+14 from five
// aligned 16-byte loads, the entries below hi counted, the descriptor
// advanced (the new cursor's value and the one 7 later are among them).
template <int KIND>
__device__ __forceinline__ int short_visit(const C4Args& A, const int4* __restrict__ ncol4,
                                           uint32_t* cnt, int4& d, int32_t wlo, int32_t base,
                                           int32_t hi, u128_t& acc) {
  const int64_t c = d.x, e = d.y, c4 = c & ~int64_t(3);
  const int off = (int)(c - c4);
  int4 v[5];
#pragma unroll
  for (int q = 0; q < 5; q++) v[q] = ncol4[(c4 >> 2) + q];
  int32_t x[W_SHORT + 7];
#pragma unroll
  for (int j = 0; j < W_SHORT + 7; j++) {
    int32_t val;
    switch (off) {
      default: val = comp(v[j >> 2], j & 3); break;
      case 1: val = comp(v[(j + 1) >> 2], (j + 1) & 3); break;
      case 2: val = comp(v[(j + 2) >> 2], (j + 2) & 3); break;
      case 3: val = comp(v[(j + 3) >> 2], (j + 3) & 3); break;
    }
    x[j] = c + j < e ? val : INT_MAX;
  }
  int took = 0;
  uint64_t part = 0;
#pragma unroll
  for (int j = 0; j < W_SHORT; j++)
    if (x[j] < hi) {
      part += window_inc_k<KIND>(A, cnt, wlo, base, x[j]);
      took++;
    }
  acc += part;
  int32_t z = x[0], w = x[7];
#pragma unroll
  for (int j = 1; j < W_SHORT; j++)
    if (j == took) {
      z = x[j];
      w = x[j + 7];
    }
  d = make_int4((int)(c + took), (int)e, z, w);
  return took;
}

// One heavy owner per workgroup, windows of counters in LDS in rank order.
// A segment is one lower neighbour's row; its descriptor holds the cursor
// (the first entry not yet counted), the row end, and the values at the
// cursor and 7 entries after it, so the length of its visit to a window is
// known to be 0, at most 7, or more without reading the row.  Rows are read
// with 16-byte loads aligned below the cursor (entries before the cursor lie
// below the window, entries from the row end on are masked; the array has
// slack after its last row).  Per pass over W_BATCH segments every thread
// first takes whole segments by itself (an empty visit costs nothing for
// descriptors held in registers, a short one five 16-byte loads); longer
// visits are queued in LDS and walked by 8-lane groups, 64 entries (two
// 16-byte loads per lane) per step, the next step's loads issued before a
// step is counted, and the next queued segment's first
// step in flight.  The next window starts at the smallest value any cursor
// points at, so windows without endpoints are never visited.
__global__ __launch_bounds__(W_NT) void k_c4_window(C4Args A) {
  constexpr int WORDS = C4_WIN_WORDS;
  constexpr int STEP = 4 * W_GL * W_LD;
  static_assert(STEP <= NCOL_PAD, "a step may read STEP entries past a cursor");
  __shared__ uint32_t cnt[WORDS];
  __shared__ int32_t queue[W_BATCH];
  __shared__ int s_item, s_q, s_minz;
  const int tid = threadIdx.x;
  const int g = tid / W_GL, gl = tid & (W_GL - 1);
  const int64_t b0 = A.start[A.bucket], cnt_items = A.start[A.bucket + 1] - b0;
  const int4* __restrict__ ncol4 = reinterpret_cast<const int4*>(A.ncol);
  const int4 kNone = make_int4(0, 0, INT_MAX, INT_MAX);
  u128_t acc = 0;
  unsigned long long wedges = 0, owners = 0, segs = 0, visits = 0;
  // counters start at zero; every window clears the words it used
  for (int i = tid; i < WORDS; i += W_NT) cnt[i] = 0;
  for (;;) {
    if (tid == 0) s_item = (int)atomicAdd(A.work, 1u);
    __syncthreads();
    const int64_t item = s_item;
    __syncthreads();
    if (item >= cnt_items) break;
    // heaviest owners (highest ranks) first
    const int64_t pos = cnt_items - 1 - item;
    const int32_t u = A.order[b0 + pos];
    const int64_t so = A.seg_off[pos];
    const int nl = A.seg_cnt[pos];
    int4* D = A.desc + so;
    // owners with at most W_BATCH segments keep each thread's descriptors in
    // registers from window to window
    const bool resident = nl <= W_BATCH;
    int4 rdesc[W_RPT];
    uint32_t stale = (1u << W_RPT) - 1u;
    if (tid == 0) {
      owners++;
      segs += (unsigned long long)nl;
    }
    const int32_t uwords = zone_words(A, u);
    int32_t wlo = 0;
    while (wlo < uwords) {
      // ranks past the last word of a zone map beyond the owner: hi = u
      const int32_t hnext = wlo + WORDS >= uwords ? u : zone_rank(A, wlo + WORDS);
      const int32_t hi = (int32_t)(hnext < u ? hnext : u);
      if (tid == 0) {
        visits += (unsigned long long)nl;
        s_minz = INT_MAX;
      }
      // the window's zone: one zone lets the counter index skip the zone tests
      const int32_t wr = zone_rank(A, wlo);
      const int kind = hi <= A.z1 ? 0 : (wr >= A.z1 && hi <= A.z2 ? 1 : (wr >= A.z2 ? 2 : 3));
      const int32_t base = wr;
      auto pass = [&](auto kind_tag) {
        constexpr int KIND = decltype(kind_tag)::value;
        for (int s0 = 0; s0 < nl; s0 += W_BATCH) {
          const int s1 = s0 + W_BATCH < nl ? s0 + W_BATCH : nl;
          if (tid == 0) s_q = 0;
          __syncthreads();
          // ---- whole segments per thread
          int32_t zmin = INT_MAX;
          if (resident) {
            // descriptors stay in registers across windows; one that a group
            // advances (a long visit) is stored before and reloaded after
#pragma unroll
            for (int j = 0; j < W_RPT; j++) {
              const int sg = tid + j * W_NT;
              if (sg < nl) {
                if ((stale >> j) & 1u) {
                  rdesc[j] = D[sg];
                  stale &= ~(1u << j);
                }
                if (rdesc[j].z < hi && rdesc[j].w < hi) {
                  D[sg] = rdesc[j];
                  queue[atomicAdd(&s_q, 1)] = sg;
                  stale |= 1u << j;
                } else {
                  if (rdesc[j].z < hi)
                    wedges += short_visit<KIND>(A, ncol4, cnt, rdesc[j], wlo, base, hi, acc);
                  zmin = min(zmin, rdesc[j].z);
                }
              }
            }
          } else {
            for (int sg = s0 + tid; sg < s1; sg += W_NT) {
              int4 d = D[sg];
              if (d.z < hi && d.w < hi) {  // 8 entries or more: queue it
                queue[atomicAdd(&s_q, 1)] = sg;
                continue;
              }
              if (d.z < hi) {
                wedges += short_visit<KIND>(A, ncol4, cnt, d, wlo, base, hi, acc);
                D[sg] = d;
              }
              zmin = min(zmin, d.z);
            }
          }
          if (zmin != INT_MAX) atomicMin(&s_minz, zmin);
          __syncthreads();
          // ---- queued long segments, one 8-lane group each: a step reads the
          // STEP entries [p, p + STEP); lane gl holds entries
          // 4 (W_GL k + gl) + r (k < W_LD, r < 4) of the step
          const int nq = s_q;
          int qi = g;
          int4 dA = qi < nq ? D[queue[qi]] : kNone;
          int64_t pA = (int64_t)dA.x & ~int64_t(STEP - 1);
          int4 a[W_LD];
#pragma unroll
          for (int k = 0; k < W_LD; k++)
            a[k] = qi < nq ? ncol4[(pA >> 2) + W_GL * k + gl] : make_int4(0, 0, 0, 0);
          while (qi < nq) {  // uniform in the group
            const int sg = queue[qi];
            const int qn = qi + W_NG;
            const int4 dB = qn < nq ? D[queue[qn]] : kNone;
            const int64_t pB = (int64_t)dB.x & ~int64_t(STEP - 1);
            int4 bn[W_LD];
#pragma unroll
            for (int k = 0; k < W_LD; k++)
              bn[k] = qn < nq ? ncol4[(pB >> 2) + W_GL * k + gl] : make_int4(0, 0, 0, 0);
            // positions fit 32 bits: the column array holds < 2^31 - 1024 entries
            const int32_t c0 = dA.x, e = dA.y;
            int32_t p = (int32_t)pA;
            int32_t cend = c0;  // new cursor
            for (;;) {
              // the next step's loads go out before this step's counting
              const bool more = p + STEP < e;
              int4 nx[W_LD];
#pragma unroll
              for (int k = 0; k < W_LD; k++)
                nx[k] = more ? ncol4[((p + STEP) >> 2) + W_GL * k + gl] : make_int4(0, 0, 0, 0);
              int mine = 0;
              // counts of one-zone windows of 4- or 8-bit counters sum below
              // 2^32 over a step; wider ones need 64 bits
              std::conditional_t<(KIND <= 1), uint32_t, uint64_t> part = 0;
              // the step's entries from the cursor on and before the row end,
              // as a bit mask over this lane's 4 W_LD entries
              const int lo_o = c0 > p ? c0 - p : 0;
              const int hi_o = e - p < STEP ? e - p : STEP;
              uint32_t pm = 0;
#pragma unroll
              for (int k = 0; k < W_LD; k++) {
                const int b = 4 * (W_GL * k + gl);
                const int lk = min(max(lo_o - b, 0), 4), hk = min(max(hi_o - b, 0), 4);
                pm |= ((1u << hk) - (1u << lk)) << (4 * k);  // lo_o <= hi_o, so lk <= hk
              }
#pragma unroll
              for (int k = 0; k < W_LD; k++)
#pragma unroll
                for (int r = 0; r < 4; r++) {
                  const int32_t xv = comp(a[k], r);
                  if (((pm >> (4 * k + r)) & 1u) && xv < hi) {
                    part += window_inc_k<KIND>(A, cnt, wlo, base, xv);
                    mine++;
                  }
                }
              acc += (uint64_t)part;
              wedges += (unsigned long long)mine;
              // entries in the window form a run from the cursor: its length is
              // the group's total
              int tot = mine;
#pragma unroll
              for (int o = 1; o < W_GL; o <<= 1) tot += __shfl_xor(tot, o, WAVE);
              const int32_t first = p > c0 ? p : c0;
              cend = first + tot;
              if (cend < p + STEP || !more) break;  // the run ends in this step
              p += STEP;
#pragma unroll
              for (int k = 0; k < W_LD; k++) a[k] = nx[k];
            }
            if (gl == 0) {
              const int32_t vnext = row_at(A.ncol, cend, e);
              D[sg] = make_int4((int)cend, (int)e, vnext, row_at(A.ncol, cend + 7, e));
              atomicMin(&s_minz, vnext);
            }
            qi = qn;
            dA = dB;
            pA = pB;
#pragma unroll
            for (int k = 0; k < W_LD; k++) a[k] = bn[k];
          }
          __syncthreads();
        }
      };
      switch (kind) {
        case 0: pass(std::integral_constant<int, 0>{}); break;
        case 1: pass(std::integral_constant<int, 1>{}); break;
        case 2: pass(std::integral_constant<int, 2>{}); break;
        default: pass(std::integral_constant<int, 3>{}); break;
      }
      // clear the counters; the next window starts at the word of the
      // smallest value a cursor points at
      const int32_t minz = s_minz;
      const int used = uwords - wlo < WORDS ? uwords - wlo : WORDS;
      for (int i = tid; i < used; i += W_NT) cnt[i] = 0;
      __syncthreads();
      wlo = minz >= u ? uwords : zone_word(A, minz);
    }
  }
  block_add_acc<W_NT>(A.scal, ACC_C4, acc);
  if (A.flags & M4_STATS) {
    block_add_u64<W_NT>(&A.scal->stat[ST_WEDGES], wedges);
    block_add_u64<W_NT>(&A.scal->kstat[A.slot][0], wedges);
    block_add_u64<W_NT>(&A.scal->kstat[A.slot][1], owners);
    block_add_u64<W_NT>(&A.scal->kstat[A.slot][2], segs);
    block_add_u64<W_NT>(&A.scal->kstat[A.slot][3], visits);
  }
}

inline unsigned blocks_for(int64_t n, int nt) { return (unsigned)ceil_div(n > 0 ? n : 1, nt); }

}  // namespace

C4Work c4_work(const Prep& P, Arena& tmp) {
  const int64_t n = P.n;
  C4Work w{};
  w.wub = tmp.take<int2>(n);
  w.key = tmp.take<uint32_t>(n);
  w.order = tmp.take<int32_t>(n);
  w.rtmp = tmp.take<int64_t>(radix_tmp_elems(n, C4_KEY_BITS));
  w.hlen = tmp.take<int32_t>(n);
  w.hoff = tmp.take<int64_t>(n + 2);
  w.stmp = tmp.take<int64_t>(scan_tmp_elems(n));
  if (!P.row_len) w.vmeta = tmp.take<int4>(n);
  if (!w.wub || !w.key || !w.order || !w.rtmp || !w.hlen || !w.hoff || !w.stmp ||
      (!P.row_len && !w.vmeta))
    throw Fail(M4_EINTERNAL, "workspace too small (c4)");
  return w;
}

void c4_enqueue(const Prep& P, const Classes& C, Scal* scal, const Tuning& tu, const C4Work& w,
                hipStream_t s, bool credit, KTimer* kt) {
  const int64_t n = P.n;
  if (n == 0 || P.m == 0) return;
  if (kt) kt->begin(M4_K_C4_PLAN, s);
  if (P.row_len) fill_u32(&scal->work_c4[0], 0, 8, s);  // one of several plans
  const C4Plan pl =
      c4_plan_rule(n, tu, scal->small.c4_start + C4_START_SLOTS, C.r1, credit);
  // rows by degree: <= 64 with 8 lanes, <= 4096 with a wavefront, longer
  // rows with a workgroup
  const int64_t b64 = C.bound[4], b4096 = C.bound[7];
  if (b64 > 0)
    k_c4_plan<8><<<blocks_for(b64 * 8, 256), 256, 0, s>>>(
        P.nptr, P.ncol, P.dr, P.dlo, 0, b64, C.r1, pl, w.wub, w.key, P.own_lo, P.hi());
  if (b4096 > b64)
    k_c4_plan<64><<<blocks_for((b4096 - b64) * 64, 256), 256, 0, s>>>(
        P.nptr, P.ncol, P.dr, P.dlo, b64, b4096, C.r1, pl, w.wub, w.key, P.own_lo, P.hi());
  if (n > b4096)
    k_c4_plan_big<<<(unsigned)(n - b4096), 1024, 0, s>>>(
        P.nptr, P.ncol, P.dr, P.dlo, b4096, C.r1, pl, w.wub, w.key, P.own_lo, P.hi());
  radix_pass(w.key, nullptr, n, 0, C4_KEY_BITS, nullptr, w.order, w.rtmp, scal->small.c4_start, s);
}

Launch c4_plan(const Prep& P, const Classes& C, Scal* scal, const Tuning& tu, uint32_t flags,
               const C4Work& w, hipStream_t s, int num_cu, KTimer* kt,
               const std::function<char*(size_t)>& big_scratch, const SmallInfo& si, bool* binned,
               unsigned long long* n8) {
  const int64_t n = P.n;
  if (n == 0 || P.m == 0) return [](hipStream_t) {};
  int2* wub = w.wub;
  int32_t* order = w.order;
  const int64_t* start = scal->small.c4_start;
  int32_t* hlen = w.hlen;
  int64_t* hoff = w.hoff;
  int64_t* stmp = w.stmp;
  int4* vmeta = w.vmeta;
  const bool small = n <= SMALL_N && !P.row_len;  // direct counters above the tiny bound
  if (kt && small) kt->begin(M4_K_C4_PLAN, s);
  std::array<int64_t, C4_START_SLOTS + 2> hstart;
  memcpy(hstart.data(), si.c4_start, sizeof(int64_t) * hstart.size());
  // counter zones of the window owners
  const int64_t z1 = std::max<int64_t>(hstart[C4_START_SLOTS], C.r1);
  const int64_t z2 = std::max<int64_t>(hstart[C4_START_SLOTS + 1], z1);
  const int64_t aw = (z1 - C.r1 + 7) >> 3, bw = (z2 - z1 + 3) >> 2;
  auto owners = [&hstart](int b) { return hstart[b + 1] - hstart[b]; };
  const int64_t HW = small ? 0 : owners(CB_WIN);
  // a partition takes whole owners: it does not hold the degrees' prefix sums
  const int64_t HB = small || P.row_len ? 0 : hstart[CB_WIDE + 1] - hstart[CB_BIN];
  if (binned) *binned = !small && hstart[CB_WIDE + 1] > hstart[CB_BIN];
  int4* desc = nullptr;
  int32_t* seg_cnt = nullptr;
  int4* parts = nullptr;
  std::array<int64_t, 3> pfirst{0, 0, 0};  // first parts of the two buckets, their end
  if (HW + HB > 0) {
    k_c4_heavy_len<<<blocks_for(HW + HB, 256), 256, 0, s>>>(order, start, P.dlo, wub, HW + HB,
                                                           hlen);
    int64_t* poff = hoff + HW + 1;
    scan_i32(hlen, HW, hoff, stmp, s);
    scan_i32(hlen + HW, HB, poff, stmp, s);
    int64_t nseg = 0;
    M4_HIP(hipMemcpyAsync(&nseg, hoff + HW, 8, hipMemcpyDeviceToHost, s));
    if (HB > 0) {
      for (int b = CB_BIN; b <= CB_WIDE; b++)
        M4_HIP(hipMemcpyAsync(&pfirst[b + 1 - CB_BIN], poff + hstart[b + 1] - hstart[CB_BIN], 8,
                              hipMemcpyDeviceToHost, s));
    }
    M4_HIP(hipStreamSynchronize(s));
    auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
    const size_t db = al((size_t)(nseg > 0 ? nseg : 1) * sizeof(int4));
    const size_t cb = al((size_t)std::max<int64_t>(HW, 1) * 4);
    const size_t pb = HB > 0 ? al((size_t)pfirst[2] * sizeof(int4)) : 0;
    char* scr = big_scratch(db + cb + pb);
    if (!scr) throw Fail(M4_ENOMEM, "no room for 4-cycle segment descriptors");
    desc = reinterpret_cast<int4*>(scr);
    seg_cnt = reinterpret_cast<int32_t*>(scr + db);
    if (HB > 0) {
      parts = reinterpret_cast<int4*>(scr + db + cb);
      k_c4_parts<<<blocks_for(pfirst[2], 256), 256, 0, s>>>(
          order + hstart[CB_BIN], wub, P.nptr, poff, HB, pfirst[2], C.r1, parts);
    }
  }
  if (kt) kt->end(M4_K_C4_PLAN, s);

  C4Args A{};
  A.order = order;
  A.start = start;
  A.nptr = P.nptr;
  A.ncol = P.ncol;
  A.dr = P.dr;
  A.dlo = P.dlo;
  A.wub = wub;
  A.row_len = P.row_len;
  A.r1 = C.r1;
  A.scal = scal;
  A.flags = flags;
  A.seg_off = hoff;
  A.desc = desc;
  A.seg_cnt = seg_cnt;
  A.vmeta = vmeta;
  A.n8 = n8;
  A.z1 = (int32_t)z1;
  A.z2 = (int32_t)z2;
  A.aw = (int32_t)aw;
  A.bw = (int32_t)bw;
  A.zr1 = (int32_t)C.r1;
  // everything below runs on the launch stream, after the plan above
  return [=](hipStream_t ls) mutable {
    if (hstart[CB_N] == hstart[CB_TINY]) return;  // no owner at all
    // with stored prefixes only the partition's rows are valid: no full pass
    if (kt) kt->begin(M4_K_C4_DESC, ls);
    if (!P.row_len && !small)
      k_vmeta<<<blocks_for(n, 256), 256, 0, ls>>>(P.nptr, P.ncol, P.dr, P.dlo, n, C.r1, vmeta);
    if (HW > 0)
      k_c4_desc<<<(unsigned)HW, 256, 0, ls>>>(order, start, hoff, P.nptr, P.dlo, P.ncol, vmeta,
                                              P.row_len, C.r1, desc, seg_cnt);
    if (kt) kt->end(M4_K_C4_DESC, ls);
    // light and tiny owners share a slot, whose one pair of events is put
    // around both kernels
    const bool hash = hstart[CB_HASH + 1] > hstart[CB_TINY];
    auto run = [&](int bucket, int slot, int hb, auto&& kernel, int nt, int64_t most, int grab) {
      int64_t cnt = hstart[bucket + 1] - hstart[bucket];
      if (cnt <= 0) return;
      A.parts = nullptr;
      if (parts && bucket >= CB_BIN) {
        A.parts = parts + pfirst[bucket - CB_BIN];
        A.npart = cnt = pfirst[bucket - CB_BIN + 1] - pfirst[bucket - CB_BIN];
      }
      A.bucket = bucket;
      A.slot = slot;
      A.work = &scal->work_c4[bucket];
      A.yb = c4_key_bits(n, hb);
      A.class_cap = bucket == CB_BIN || bucket == CB_WIDE ? tu.c4_bin_cap : 0;
      A.grab = grab;
      const bool timed = kt && slot != M4_K_C4_HASH;
      if (timed) kt->begin(slot, ls);
      kernel<<<(unsigned)std::min<int64_t>(most, ceil_div(cnt, grab)), nt, 0, ls>>>(A);
      if (timed) kt->end(slot, ls);
    };
    auto filter = [&](int bucket, int slot, int hb, auto&& plain, auto&& cred, int nt,
                      int per_cu) {
      run(bucket, slot, hb, n8 ? cred : plain, nt, (int64_t)num_cu * per_cu, 1);
    };
    const int64_t waves = (int64_t)num_cu * 32;
    if (small) {
      // the owners of every bucket above the tiny one: a kernel for all
      hstart[CB_HASH + 1] = hstart[CB_N];
      if (kt) kt->begin(M4_K_C4_HASH, ls);
      filter(CB_HASH, M4_K_C4_HASH, 1, k_c4_direct<false>, k_c4_direct<true>, 256, 4);
      run(CB_TINY, M4_K_C4_HASH, 1, n8 ? k_c4_tiny<true> : k_c4_tiny<false>, WAVE, waves, 1);
      if (kt) kt->end(M4_K_C4_HASH, ls);
      return;
    }
    // heavy owners first
    if (n8)
      run(CB_WIDE, M4_K_C4_BIN, C4_BIN_AB - 7,
          k_c4_filter<1024, 16, C4_BIN_AB - 1, C4_BIN_BB, 512, true, true>, 1024, num_cu, 1);
    filter(CB_BIN, M4_K_C4_BIN, C4_BIN_AB - 5,
           k_c4_filter<1024, 8, C4_BIN_AB, C4_BIN_BB, 512, false>,
           k_c4_filter<1024, 8, C4_BIN_AB, C4_BIN_BB, 512, true>, 1024, 1);
    run(CB_WIN, M4_K_C4_WINDOW, 1, k_c4_window, W_NT, num_cu, 1);
    filter(CB_MED, M4_K_C4_MED, C4_MED_AB - 5,
           k_c4_filter<256, 8, C4_MED_AB, C4_MED_BB, 128, false>,
           k_c4_filter<256, 8, C4_MED_AB, C4_MED_BB, 128, true>, 256, 6);
    if (kt && hash) kt->begin(M4_K_C4_HASH, ls);
    filter(CB_HASH, M4_K_C4_HASH, C4_LIGHT_AB - 5,
           k_c4_filter<64, 8, C4_LIGHT_AB, C4_LIGHT_BB, 64, false>,
           k_c4_filter<64, 8, C4_LIGHT_AB, C4_LIGHT_BB, 64, true>, 64, 24);
    // a wavefront takes up to 16 owners at once where that still fills the
    // device (32 wavefronts a CU), fewer where it would not
    const int64_t tiny = hstart[CB_TINY + 1] - hstart[CB_TINY];
    run(CB_TINY, M4_K_C4_HASH, 1, n8 ? k_c4_tiny<true> : k_c4_tiny<false>, WAVE, waves,
        (int)std::max<int64_t>(1, std::min<int64_t>(16, tiny / waves)));
    if (kt && hash) kt->end(M4_K_C4_HASH, ls);
  };
}

}  // namespace m4
