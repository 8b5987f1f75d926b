// m4_walk_dev.h -- walks over sorted row segments by groups of lanes, and the
// per-wavefront queue that gathers the few entries a walk is after.
#pragma once
#include <limits.h>

#include "m4_device.h"

namespace m4 {

// Walks the entries below hi of segments [0, nseg): groups of GL lanes take
// segments one at a time from *next (LDS, zero at the start), a step being
// 4 GL entries as one aligned 16-byte load per lane.  A group that meets an
// entry >= hi or the segment's end (both show in its last lane: entries
// ascend, and the lanes past the end count as ended) takes its next segment
// before it works on the step, so the following load is always in flight.
// One LDS atomic per wavefront serves all of its groups that end in a step.
// seg(i) gives {first entry, end} of segment i, an empty one at i = nseg (held
// by the groups without a segment).  The per-entry tests stay in vector registers (one unsigned compare for the segment, one
// for hi): a version with lane-mask logic was bound by the scalar unit.
//   ent(x, i, at)  the lane's four entries, INT_MAX where not of the segment
//                  (an entry counts when it is below hi), its segment and the
//                  place of the first entry in ncol
//   fin(i, last)   after a step, by every lane of the wavefront; last is set
//                  in the groups whose segment i (i < nseg) ended with it
template <int GL, class Seg, class Ent, class Fin>
__device__ __forceinline__ void seg_walk(const int32_t* __restrict__ ncol, int32_t hi, int nseg,
                                         int* next, Seg&& seg, Ent&& ent, Fin&& fin) {
  static_assert(4 * GL <= NCOL_PAD, "a step may read 4 GL entries past a cursor");
  const int lane = threadIdx.x & (WAVE - 1), gl = lane & (GL - 1);
  constexpr uint64_t LASTS = GL == 8 ? 0x8080808080808080ull : 0x8000800080008000ull;
  static_assert(GL == 8 || GL == 16, "a group is 8 or 16 lanes");
  const int4* __restrict__ ncol4 = reinterpret_cast<const int4*>(ncol);
  // indices for the groups whose last lane is set in m (nonzero, uniform):
  // a lane's value is its own group's when that is among them
  auto grab = [&](uint64_t m) {
    int b = 0;
    if (lane == 0) b = atomicAdd(next, (int)__popcll(m));
    return __builtin_amdgcn_readfirstlane(b) +
           (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
  };
  int i = min(grab(LASTS), nseg);
  int2 s = seg(i);
  int q4 = (s.x >> 2) + gl;           // the lane's 16-byte load
  int off = (q4 << 2) - s.x;          // its first entry's place in the segment
  int len = s.y - s.x;
  int4 a = ncol4[q4];
  while (__ballot(i < nseg)) {
    const uint64_t ended = __ballot(max(a.w - hi, off + 4 - len) >= 0) & LASTS;
    const int sh = lane | (GL - 1);
    const bool last = (((sh < 32 ? (uint32_t)ended : (uint32_t)(ended >> 32)) >> (sh & 31)) & 1) != 0;
    int ni = i, nq4 = q4 + GL, noff = off + 4 * GL, nlen = len;
    if (ended) {
      const int g = min(grab(ended), nseg);
      const int2 t = seg(g);
      const int t4 = (t.x >> 2) + gl;
      ni = last ? g : ni;
      nq4 = last ? t4 : nq4;
      noff = last ? (t4 << 2) - t.x : noff;
      nlen = last ? t.y - t.x : nlen;
    }
    const int4 nx = ncol4[nq4];
    const int32_t x[4] = {(unsigned)off < (unsigned)len ? a.x : INT_MAX,
                          (unsigned)(off + 1) < (unsigned)len ? a.y : INT_MAX,
                          (unsigned)(off + 2) < (unsigned)len ? a.z : INT_MAX,
                          (unsigned)(off + 3) < (unsigned)len ? a.w : INT_MAX};
    ent(x, i, q4 << 2);
    fin(i, last && i < nseg);
    i = ni;
    q4 = nq4;
    off = noff;
    len = nlen;
    a = nx;
  }
}

// Lanes below this one among the set lanes of m.
__device__ __forceinline__ int lanes_before(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                        __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

}  // namespace m4
