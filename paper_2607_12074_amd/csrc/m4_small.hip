// m4_small.hip -- preparation and plan of small graphs (at most SMALL_N
// vertices) in three kernels and one read-back.
//
// A call on a graph of a few thousand vertices is bound by its launches and
// read-backs (4-5 us of host time each, 10 us and more for a read-back), not by
// its work.  The general path takes about 30 launches and 5 read-backs to order
// the vertices, sort the rows by degree class, price the anchor bases and
// bucket the owners of both anchor stages.  Here the degree order fits the LDS
// of one workgroup and a row is a bitmap of at most SMALL_N bits, so
//   k_small_order  (one workgroup) sorts by degree: perm, rank, dr, row offsets,
//                  class and zone bounds;
//   k_small_rows   relabels and sorts the rows through LDS bitmaps and takes
//                  along what needs the neighbours' degrees;
//   k_small_plan   (two workgroups) the oriented offsets and out-list records,
//                  hub tables and buckets of the triangle owners; the buckets of
//                  the 4-cycle owners and the inputs of the anchor objective.
// Whole calls, us, general path / this one: 2000 vertices and 20000 edges
// 353 / 114, 5000 vertices of a power law from host arrays 440 / 176, per-vertex
// orbits of the first 351 / 161.  The bound is the LDS of k_small_order (two
// buffers of SMALL_N keys) and the rows' bitmap (four words a lane).
#include <algorithm>

#include "m4_plan_dev.h"
#include "m4_tri_dev.h"
#include "m4_walk_dev.h"

namespace m4 {

namespace {

constexpr int SM_NT = 1024, SM_NW = SM_NT / WAVE;
constexpr int SM_BITS = 13, SM_WORDS = SMALL_N / 32;
static_assert(SMALL_N == 1 << SM_BITS, "a degree and an id share a sort key");
constexpr int SM_DIG = 7;  // digit of a sort pass
constexpr int SM_LONG = 256, SM_LONG_AT = 5;  // longer rows take a workgroup; Classes::bound[]

struct SmallThr {
  int thr[16];
  int n;
};

// Stable LSD sort of (degree, id) by degree: every wavefront keeps its own
// digit counters over its run of the vertices, so the passes need no atomics
// and three barriers each; an item's place among its wavefront's equal digits
// is kept in a register from counting to placing (5000 vertices, two passes:
// 30 us when found twice, 26 so).  Degrees are clamped to the key's bits (a simple
// graph has none beyond).
__global__ __launch_bounds__(SM_NT) void k_small_order(const int64_t* __restrict__ rp, int n,
                                                       SmallThr T, bool zero,
                                                       int32_t* __restrict__ perm,
                                                       int32_t* __restrict__ rank,
                                                       int32_t* __restrict__ dr,
                                                       int64_t* __restrict__ nptr, Scal* scal) {
  __shared__ uint32_t kb[2][SMALL_N];
  __shared__ int cnt[SM_NW << SM_DIG];
  __shared__ int s_dmax;
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid / WAVE;
  if (zero)
    for (int i = tid; i < (int)(sizeof(Scal) / 4); i += SM_NT)
      reinterpret_cast<uint32_t*>(scal)[i] = 0;
  if (tid == 0) s_dmax = 0;
  __syncthreads();
  int dm = 0;
  for (int i = tid; i < n; i += SM_NT) {
    const int64_t d64 = rp[i + 1] - rp[i];
    const int d = d64 < 0 ? 0 : (d64 < SMALL_N ? (int)d64 : SMALL_N - 1);
    kb[0][i] = (uint32_t)d << SM_BITS | (uint32_t)i;
    dm = max(dm, d);
  }
  if (dm) atomicMax(&s_dmax, dm);
  __syncthreads();
  const int dmax = s_dmax;
  const int run = (n + SM_NW * WAVE - 1) / (SM_NW * WAVE) * WAVE;  // vertices of a wavefront
  const int lo = w * run, hi = min(n, lo + run);
  const uint32_t* src = kb[0];
  uint32_t* dst = kb[1];
  for (int shift = 0; shift < SM_BITS && (shift == 0 || dmax >> shift); shift += SM_DIG) {
    for (int i = tid; i < SM_NW << SM_DIG; i += SM_NT) cnt[i] = 0;
    __syncthreads();
    // count, keeping each item's place among its wavefront's equal digits
    constexpr int STEPS = SMALL_N / SM_NT;
    uint32_t key[STEPS];
    int place[STEPS];
#pragma unroll
    for (int q = 0; q < STEPS; q++) {
      const int i0 = lo + q * WAVE;
      if (i0 >= hi) break;
      const bool valid = i0 + lane < hi;
      key[q] = valid ? src[i0 + lane] : 0;
      const int dig = (key[q] >> (SM_BITS + shift)) & ((1 << SM_DIG) - 1);
      uint64_t same = __ballot(valid);
#pragma unroll
      for (int b = 0; b < SM_DIG; b++) {
        const uint64_t m = __ballot((dig >> b) & 1);
        same &= (dig >> b) & 1 ? m : ~m;
      }
      const int before = lanes_before(same);
      const int at = cnt[w << SM_DIG | dig];
      wave_sync();
      place[q] = at + before;
      if (valid && before == 0) cnt[w << SM_DIG | dig] = at + (int)__popcll(same);
      wave_sync();
    }
    __syncthreads();
    {
      constexpr int PER = (SM_NW << SM_DIG) / SM_NT;
      int c[PER], s = 0;
#pragma unroll
      for (int k = 0; k < PER; k++) {
        const int e = tid * PER + k;  // by digit, then wavefront
        c[k] = cnt[(e % SM_NW) << SM_DIG | e / SM_NW];
        s += c[k];
      }
      int at = (int)block_excl_scan64<SM_NT>(s, nullptr);
#pragma unroll
      for (int k = 0; k < PER; k++) {
        const int e = tid * PER + k;
        cnt[(e % SM_NW) << SM_DIG | e / SM_NW] = at;
        at += c[k];
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < STEPS; q++)
      if (lo + q * WAVE + lane < hi)
        dst[place[q] + cnt[w << SM_DIG | ((key[q] >> (SM_BITS + shift)) & ((1 << SM_DIG) - 1))]] =
            key[q];
    __syncthreads();
    const uint32_t* t = src;
    src = dst;
    dst = const_cast<uint32_t*>(t);
  }
  const int per = (n + SM_NT - 1) / SM_NT;
  const int r0 = min(n, tid * per), r1 = min(n, r0 + per);
  int64_t s = 0, tot;
  for (int r = r0; r < r1; r++) s += src[r] >> SM_BITS;
  int64_t at = block_excl_scan64<SM_NT>(s, &tot);
  for (int r = r0; r < r1; r++) {
    const int d = (int)(src[r] >> SM_BITS), id = (int)(src[r] & (SMALL_N - 1));
    perm[r] = id;
    rank[id] = r;
    dr[r] = d;
    nptr[r] = at;
    at += d;
  }
  if (tid == 0) {
    nptr[n] = tot;
    scal->small.dmax = dmax;
    scal->dmax = (unsigned)dmax;
  }
  // first rank of a larger degree than each class threshold, and than the two
  // of the 4-cycle counter zones
  if (tid < T.n + 2) {
    const int thr = tid < T.n ? T.thr[tid] : (tid == T.n ? 15 : 255);
    int a = 0, b = n;
    while (a < b) {
      const int mid = (a + b) >> 1;
      if ((int)(src[mid] >> SM_BITS) <= thr) a = mid + 1;
      else b = mid;
    }
    if (tid < T.n) scal->small.bound[tid] = a;
    else scal->small.c4_start[C4_START_SLOTS + tid - T.n] = a;
  }
}

struct SmallRow {
  const int64_t* rp;
  const int32_t* col;
  const int32_t* perm;
  const int32_t* rank;
  const int32_t* dr;
  const int64_t* nptr;
  int32_t* ncol;
  int32_t* dlo;
  int32_t* dplus;
  int2* wub;       // {wedge bound, lower neighbours of degree above 1}; the bound is the
                   // sum of (degree - 1) over the lower neighbours
  int4* vmeta;     // {row offset, degree, lower neighbours, entries below r1}
  int64_t* dsum;   // sum of the neighbours' degrees
  uint32_t* t;
  int64_t m;
  const int64_t* bound;  // Classes::bound
  int n;
};

// A wavefront per row: the entries' ranks set bits of an LDS bitmap, which is
// read back in order; rows of more than SM_LONG entries take a workgroup of the
// SM_LONG_BLOCKS behind the others'.  Entries that are in a row twice (no simple
// graph) are followed by the largest rank, so that every place is written.
constexpr int SM_ROW_NT = 256, SM_LONG_BLOCKS = 256;
__global__ __launch_bounds__(SM_ROW_NT) void k_small_rows(SmallRow A) {
  constexpr int NW = SM_ROW_NT / WAVE;
  __shared__ uint4 bm4[NW][SM_WORDS / 4];
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid / WAVE;
  for (int64_t i = (int64_t)blockIdx.x * SM_ROW_NT + tid; i < A.m;
       i += (int64_t)gridDim.x * SM_ROW_NT)
    A.t[i] = 0;
  const int r1 = (int)A.bound[0], rlong = (int)A.bound[SM_LONG_AT];
  const int row_blocks = (A.n + NW - 1) / NW;
  static_assert(SM_WORDS == 4 * WAVE && SM_WORDS == SM_ROW_NT, "words of a lane and of a thread");
  if ((int)blockIdx.x < row_blocks) {
    const int r = blockIdx.x * NW + w;
    if (r >= rlong || r >= A.n) return;
    uint32_t* bm = reinterpret_cast<uint32_t*>(bm4[w]);
    bm4[w][lane] = make_uint4(0, 0, 0, 0);
    const int d = A.dr[r];
    const int64_t in0 = A.rp[A.perm[r]], out0 = A.nptr[r];
    wave_sync();
    int below = 0, cut = 0, wb = 0, ds = 0;
    int32_t x[SM_LONG / WAVE];
#pragma unroll
    for (int q = 0; q < SM_LONG / WAVE; q++) {
      const int i = q * WAVE + lane;
      x[q] = i < d ? A.rank[A.col[in0 + i]] : -1;
    }
#pragma unroll
    for (int q = 0; q < SM_LONG / WAVE; q++) {
      if (x[q] < 0) continue;
      atomicOr(&bm[x[q] >> 5], 1u << (x[q] & 31));
      const int dx = A.dr[x[q]];
      below += x[q] < r;
      cut += x[q] < r1;
      wb += x[q] < r ? dx - 1 : 0;
      ds += dx;
    }
    wave_sync();
    const uint4 v = bm4[w][lane];
    const uint32_t word[4] = {v.x, v.y, v.z, v.w};
    const int mine = __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
    int at = mine;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const int y = __shfl_up(at, o, WAVE);
      if (lane >= o) at += y;
    }
    const int have = __shfl(at, WAVE - 1, WAVE);
    at -= mine;
    int32_t* out = A.ncol + out0;
#pragma unroll
    for (int k = 0; k < 4; k++) {
      uint32_t bits = word[k];
      while (bits) {
        out[at++] = (4 * lane + k) * 32 + __ffs(bits) - 1;
        bits &= bits - 1;
      }
    }
    for (int i = have + lane; i < d; i += WAVE) out[i] = A.n - 1;
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) {
      below += __shfl_xor(below, o, WAVE);
      cut += __shfl_xor(cut, o, WAVE);
      wb += __shfl_xor(wb, o, WAVE);
      ds += __shfl_xor(ds, o, WAVE);
    }
    if (lane == 0) {
      A.dlo[r] = below;
      A.dplus[r] = d - below;
      A.wub[r] = make_int2(wb, below - min(cut, below));
      A.dsum[r] = ds;
      A.vmeta[r] = make_int4((int)out0, d, below, cut);
    }
    return;
  }
  uint32_t* bm = reinterpret_cast<uint32_t*>(bm4[0]);
  for (int r = rlong + ((int)blockIdx.x - row_blocks); r < A.n; r += SM_LONG_BLOCKS) {
    bm[tid] = 0;
    const int d = A.dr[r];
    const int64_t in0 = A.rp[A.perm[r]], out0 = A.nptr[r];
    __syncthreads();
    // two counts of at most 2^13 and two sums of at most 2^26 to a word
    int64_t nums = 0, sums = 0;
    for (int i = tid; i < d; i += SM_ROW_NT) {
      const int32_t x = A.rank[A.col[in0 + i]];
      atomicOr(&bm[x >> 5], 1u << (x & 31));
      const int dx = A.dr[x];
      nums += (int64_t)(x < r1) << 32 | (x < r);
      sums += (int64_t)(x < r ? dx - 1 : 0) << 32 | dx;
    }
    int64_t ntot, stot, have;
    block_excl_scan64<SM_ROW_NT>(nums, &ntot);
    block_excl_scan64<SM_ROW_NT>(sums, &stot);
    uint32_t bits = bm[tid];
    int64_t at = block_excl_scan64<SM_ROW_NT>(__popc(bits), &have);
    int32_t* out = A.ncol + out0;
    while (bits) {
      out[at++] = tid * 32 + __ffs(bits) - 1;
      bits &= bits - 1;
    }
    for (int64_t i = have + tid; i < d; i += SM_ROW_NT) out[i] = A.n - 1;
    if (tid == 0) {
      const int below = (int)(uint32_t)ntot, cut = (int)(ntot >> 32);
      A.dlo[r] = below;
      A.dplus[r] = d - below;
      A.wub[r] = make_int2((int)(stot >> 32), below - min(cut, below));
      A.dsum[r] = (uint32_t)stot;
      A.vmeta[r] = make_int4((int)out0, d, below, cut);
    }
    __syncthreads();
  }
}

struct SmallPlan {
  const int32_t* dr;
  const int32_t* dlo;
  const int32_t* dplus;
  const int64_t* nptr;
  int64_t* optr;
  int n, small_max, wave_max, hub_min;
  int32_t* tri_order;
  int2* list;
  int32_t* hoff;
  int32_t* hub_list;
  C4Plan pl;  // r1 is read on the device
  const int2* wub;
  const int64_t* dsum;
  int32_t* c4_order;
};

constexpr int PL_NT = 512;
// Stable partition of the block's items by a 3-bit key: thread t holds items
// [i0, i1), the counts of four keys share a 64-bit scan.
template <class Key>
__device__ __forceinline__ void partition8(int n, int i0, int i1, Key key, int32_t* order,
                                           int64_t* start, int slots) {
  uint64_t c[2] = {0, 0};
#pragma unroll 1
  for (int i = i0; i < i1; i++) {
    const uint32_t k = key(i);
    const uint64_t one = 1ull << (16 * (k & 3));
    c[0] += k >> 2 ? 0 : one;
    c[1] += k >> 2 ? one : 0;
  }
  int64_t ex[2], tot[2];
  ex[0] = block_excl_scan64<PL_NT>((int64_t)c[0], &tot[0]);
  ex[1] = block_excl_scan64<PL_NT>((int64_t)c[1], &tot[1]);
  __shared__ int first[8];
  if (threadIdx.x == 0) {
    int at = 0;
    for (int k = 0; k < slots; k++) {
      start[k] = at;
      if (k < 8) {
        first[k] = at;
        at += (int)((uint64_t)(k >> 2 ? tot[1] : tot[0]) >> (16 * (k & 3))) & 0xffff;
      }
    }
  }
  __syncthreads();
  uint64_t run[2] = {(uint64_t)ex[0], (uint64_t)ex[1]};
#pragma unroll 1
  for (int i = i0; i < i1; i++) {
    const uint32_t k = key(i);
    const uint64_t r = k >> 2 ? run[1] : run[0], one = 1ull << (16 * (k & 3));
    order[first[k] + ((int)(r >> (16 * (k & 3))) & 0xffff)] = i;
    run[0] += k >> 2 ? 0 : one;
    run[1] += k >> 2 ? one : 0;
  }
}

// The threads own runs of vertices, so what they read in several loops comes
// through LDS, loaded in order (5000 vertices: 21 us read in place, 18 so).
__global__ __launch_bounds__(PL_NT) void k_small_plan(SmallPlan A, Scal* scal) {
  __shared__ int32_t val[SMALL_N];  // out-degrees; 4-cycle buckets
  static_assert(SMALL_N < 1 << 16 && TK_N <= 8 && CB_N <= 8, "packed counts");
  __shared__ unsigned s_nhub, s_kmax;
  SmallInfo& S = scal->small;
  const int tid = threadIdx.x, n = A.n;
  const int per = (n + PL_NT - 1) / PL_NT;
  const int i0 = min(n, tid * per), i1 = min(n, i0 + per);
  if (blockIdx.x == 0) {
    if (tid == 0) s_nhub = s_kmax = 0;
#pragma unroll 4
    for (int i = tid; i < n; i += PL_NT) val[i] = A.dplus[i];
    __syncthreads();
    int64_t ds = 0, hs = 0, dtot, htot = 0;
    int kmax = 0;
#pragma unroll 1
    for (int i = i0; i < i1; i++) {
      const int k = val[i];
      ds += k;
      kmax = max(kmax, k);
      if (A.hoff && k >= A.hub_min) hs += 1 << hub_bits(k);
    }
    int64_t d = block_excl_scan64<PL_NT>(ds, &dtot);
    int64_t h = A.hoff ? block_excl_scan64<PL_NT>(hs, &htot) : 0;
    if (kmax > TRI_LDS_MAX) atomicMax(&s_kmax, (unsigned)kmax);
#pragma unroll 4
    for (int i = i0; i < i1; i++) {
      const int k = val[i];
      A.optr[i] = d;
      A.list[i] = make_int2((int)(A.nptr[i] + A.dlo[i]), (int)d);
      d += k;
      if (A.hoff) {
        const bool hub = k >= A.hub_min;
        A.hoff[i] = hub ? (int32_t)h : -1;
        if (hub) {
          h += 1 << hub_bits(k);
          A.hub_list[atomicAdd(&s_nhub, 1u)] = i;
        }
      }
    }
    partition8(
        n, i0, i1, [&](int i) { return tri_bucket(val[i], A.small_max, A.wave_max); },
        A.tri_order, S.tri_start, 17);
    __syncthreads();
    if (tid == 0) {
      A.optr[n] = dtot;
      A.list[n] = make_int2(0, (int)dtot);
      scal->nhub = s_nhub;
      S.kmax = s_kmax;
      S.hub_slots = htot;
    }
    return;
  }
  C4Plan pl = A.pl;
  pl.r1 = S.bound[0];
  int64_t wedge = 0, lower = 0, scan = 0;
#pragma unroll 2
  for (int i = tid; i < n; i += PL_NT) {
    const int2 wb = A.wub[i];
    val[i] = i >= pl.r1 && A.dlo[i] >= 2 && wb.x > 0 ? (int)c4_bucket(pl, wb.x, i, wb.y)
                                                     : (int)CB_NONE;
    const int64_t dg = A.dr[i], k = A.dplus[i];
    if (dg >= 2) wedge += (dg - 1) * k;
    lower += dg * k;
    scan += A.dsum[i] * k;
  }
  int64_t tw, tl, ts;  // the scans' barriers also stand between val's writes and reads
  block_excl_scan64<PL_NT>(wedge, &tw);
  block_excl_scan64<PL_NT>(lower, &tl);
  block_excl_scan64<PL_NT>(scan, &ts);
  partition8(
      n, i0, i1, [&](int i) { return (uint32_t)val[i]; }, A.c4_order, S.c4_start, C4_START_SLOTS);
  if (tid == 0) {
    S.cost[0] = (unsigned long long)tw;
    S.cost[1] = (unsigned long long)tl;
    S.cost[2] = (unsigned long long)A.dr[n - 1];
    S.cost[3] = (unsigned long long)ts;
  }
}

}  // namespace

void small_prep(const int64_t* rp, const int32_t* col, int64_t n, int64_t nnz, Prep& P, Classes& C,
                const Tuning& tu, uint32_t flags, uint32_t cache_rows, bool credit,
                const TriWork& tw, const C4Work& cw, Scal* scal, Scal* scal_host, hipStream_t s) {
  P.n = n;
  P.nnz = nnz;
  P.m = nnz / 2;
  const bool validate = (flags & M4_VALIDATE) != 0;
  if (validate) {
    fill_u32(scal, 0, sizeof(Scal) / 4, s);
    validate_csr(rp, col, n, nnz, scal, s);
    M4_HIP(hipMemcpyAsync(scal_host, scal, kScalHead, hipMemcpyDeviceToHost, s));
    M4_HIP(hipStreamSynchronize(s));
    if (scal_host->err) throw Fail(M4_EINVAL, "CSR is not simple, symmetric and sorted");
  }
  SmallThr T{};
  T.n = row_class_count();
  for (int i = 0; i < T.n; i++) T.thr[i] = row_class_thresholds()[i];
  if (T.thr[SM_LONG_AT] != SM_LONG) throw Fail(M4_EINTERNAL, "row classes changed");
  k_small_order<<<1, SM_NT, 0, s>>>(rp, (int)n, T, !validate, P.perm, P.rank, P.dr, P.nptr, scal);
  // the wedge bounds and segment offsets of the 4-cycle workspace; the latter
  // are not used by small graphs and hold the neighbours' degree sums
  const SmallRow R{rp,      col,     P.perm,   P.rank,  P.dr, P.nptr, P.ncol,            P.dlo,
                   P.dplus, cw.wub,  cw.vmeta, cw.hoff, P.t,  P.m,    scal->small.bound, (int)n};
  const unsigned long_blocks = (unsigned)std::min<int64_t>(SM_LONG_BLOCKS, nnz / SM_LONG);
  k_small_rows<<<(unsigned)ceil_div(n, SM_ROW_NT / WAVE) + long_blocks, SM_ROW_NT, 0, s>>>(R);
  SmallPlan A{};
  A.dr = P.dr;
  A.dlo = P.dlo;
  A.dplus = P.dplus;
  A.nptr = P.nptr;
  A.optr = P.optr;
  A.n = (int)n;
  tri_bounds(P, tu, flags, cache_rows, &A.small_max, &A.wave_max);
  A.hub_min = tu.hub_min;
  A.tri_order = tw.order;
  A.list = reinterpret_cast<int2*>(tw.hoff64);
  A.hoff = tw.hoff;
  A.hub_list = tw.hub_list;
  A.pl = c4_plan_rule(n, tu, scal->small.c4_start + C4_START_SLOTS, 0, credit);
  A.wub = cw.wub;
  A.dsum = cw.hoff;
  A.c4_order = cw.order;
  k_small_plan<<<2, PL_NT, 0, s>>>(A, scal);
  M4_HIP(hipMemcpyAsync(scal_host, scal, kScalHead, hipMemcpyDeviceToHost, s));
  M4_HIP(hipStreamSynchronize(s));
  const SmallInfo& S = scal_host->small;
  C.dmax = S.dmax;
  for (int i = 0; i < T.n; i++) C.bound[i] = S.bound[i];
  C.r1 = C.bound[0];
}

}  // namespace m4
