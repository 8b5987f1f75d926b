// m4_plan_dev.h -- which kernel takes an owner: the bucket rules of the
// triangle and 4-cycle stages, shared by their own plan kernels and by the
// plan of small graphs.
#pragma once
#include <limits.h>

#include "m4_device.h"

namespace m4 {

// Triangle owners by out-degree k.
enum { TK_NONE = 0, TK_WAVE, TK_128, TK_256, TK_512, TK_1024, TK_GLOBAL, TK_SMALL, TK_N };
__device__ __forceinline__ uint32_t tri_bucket(int k, int small_max, int wave_max) {
  if (k < 2) return TK_NONE;
  if (k <= small_max) return TK_SMALL;
  if (k <= wave_max) return TK_WAVE;
  if (k <= 128) return TK_128;
  if (k <= 256) return TK_256;
  if (k <= 512) return TK_512;
  return k <= TRI_LDS_MAX ? TK_1024 : TK_GLOBAL;
}

// Filtered owners: log2 of the bits of the first and second LDS bitmap of
// each bucket (the first holds 2^(bits - 5) table slots afterwards).
constexpr int C4_LIGHT_AB = 15, C4_LIGHT_BB = 13;
constexpr int C4_MED_AB = 17, C4_MED_BB = 15;
constexpr int C4_BIN_AB = 20, C4_BIN_BB = 17;
constexpr int C4_DISP_BITS = 6;                  // distance of a slot from its home slot

// Bits of a permuted rank for tables of 2^hb slots, and the first number of
// lower neighbours whose counts do not fit beside the key in a slot.
inline int c4_key_bits(int64_t n, int hb) {
  int b = hb;
  while ((int64_t(1) << b) < n) b++;
  return b;
}
inline int32_t c4_count_limit(int64_t n, int hb) {
  const int bits = 32 - C4_DISP_BITS - (c4_key_bits(n, hb) - hb);
  return bits >= 31 ? INT_MAX : (bits <= 0 ? 0 : 1 << bits);
}

// Windows of dense counters owner u needs over ranks [r1, u); zb holds the
// first ranks of degree > 15 and > 255 (the zone bounds).
__device__ __forceinline__ int64_t c4_windows(const int64_t* zb, int64_t r1, int64_t u) {
  const int64_t z1 = zb[0] > r1 ? zb[0] : r1, z2 = zb[1] > z1 ? zb[1] : z1;
  const int64_t aw = (z1 - r1 + 7) >> 3, bw = (z2 - z1 + 3) >> 2;
  int64_t words;
  if (u <= r1) words = 0;
  else if (u <= z1) words = (u - r1 + 7) >> 3;
  else if (u <= z2) words = aw + ((u - z1 + 3) >> 2);
  else words = aw + bw + (u - z2);
  return (words + C4_WIN_WORDS - 1) / C4_WIN_WORDS;
}

// Bucket of owner u with wedge bound w > 0 and nl lower neighbours of degree
// above 1.  Owners up to C4_TINY_MAX wedges take one wavefront and a table, the
// ones above a bitmap filter sized to their bound.  Beyond the one-pass medium
// bound a dense window costs a pass over the owner's lower neighbours, so an
// owner goes to the filter of the ranged medium bucket only when its endpoints
// are thin over many windows (16 windows >= med_win ranges of C4_MED_CAP
// endpoints; med_win 0: never), to the large filter when they span at least
// bin_win windows and average fewer than bin_dense endpoints per window, and
// else keeps the dense windows.  A filter needs its counts to fit beside the key
// (lower neighbours below its limit); with credits (orbit counts) there are no
// dense windows and the large filter takes the rest, or its variant with 64-bit
// slots.
struct C4Plan {
  int light_max, med_max, med_win, bin_win, bin_dense;
  const int64_t* zb;
  int64_t r1;
  int32_t lim_light, lim_med, lim_bin;
  int credit;
};
__device__ __forceinline__ uint32_t c4_bucket(const C4Plan& pl, int64_t w, int64_t u, int nl) {
  if (w <= pl.light_max) {
    if (w <= C4_TINY_MAX) return CB_TINY;
    if (nl < pl.lim_light) return CB_HASH;
  }
  if (pl.med_max > 0 && w <= pl.med_max && w <= C4_MED_CAP && nl < pl.lim_med) return CB_MED;
  const int64_t nwin = c4_windows(pl.zb, pl.r1, u);
  if (pl.bin_win > 0 && nwin >= pl.bin_win && nl < pl.lim_bin &&
      (pl.bin_dense <= 0 || w < (int64_t)pl.bin_dense * nwin))
    return CB_BIN;
  if (pl.med_max > 0 && pl.med_win > 0 && w <= C4_MED_MAX && nl < pl.lim_med &&
      16 * nwin >= (int64_t)pl.med_win * ((w + C4_MED_CAP - 1) / C4_MED_CAP))
    return CB_MED;
  if (pl.credit) return nl < pl.lim_bin ? CB_BIN : CB_WIDE;
  return CB_WIN;
}

inline C4Plan c4_plan_rule(int64_t n, const Tuning& tu, const int64_t* zb, int64_t r1,
                           bool credit) {
  return C4Plan{tu.c4_light_max, tu.c4_med_max, tu.c4_med_win, tu.c4_bin_win, tu.c4_bin_dense,
                zb, r1, c4_count_limit(n, C4_LIGHT_AB - 5), c4_count_limit(n, C4_MED_AB - 5),
                c4_count_limit(n, C4_BIN_AB - 5), credit ? 1 : 0};
}

}  // namespace m4
