// Internal: which tile a workgroup computes.  (Plain arithmetic, so that a test can go through it on the host.)
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#define S2_HD __host__ __device__
#else
#define S2_HD
#endif

namespace s2 {

// Workgroup index -> (batch*head, rank inside the head) such that all tiles of one (batch, head)
// run on one XCD.  Workgroups are handed to the 8 XCDs round-robin by linear index, and each XCD
// has its own L2: keeping a head's key/value stripes and moving window on one XCD lets every
// later query tile of that head hit in that L2.
// The pairs that are left over where their number is not a multiple of eight are shared by all XCDs: an XCD with a pair more than
// another would still be at work when that one is done.  They are dealt out in runs of tiles of following ranks, by rank, so that
// neighbouring windows still meet in an L2.  Forward and backward, us, with the left-over pairs on an XCD each and dealt out: 1 x 9 heads x 16384 x 128
// 159 and 118, 520 and 339; 3 x 8192 44 and 29, 126 and 87; 20 x 4096 35 and 33, 106 and 92; 33 x 4096 x 64 37 and 31, 92 and 79; dense 19 x
// 7168 290 and 234, 818 and 680; where seven are left over, and little is lost by an XCD each, 15 x 8192 x 128 84 and 81, 239 and 239.  (Single tiles instead of runs:
// 118 and 361, 30 and 90, 33 and 93, 32 and 79, 233 and 701, 85 and 251; at 64 tiles runs of four are 1 to 3 % slower than of two, at 128 none is.)
S2_HD inline int deal_run(int tiles) { return tiles >= 128 ? 4 : tiles >= 64 ? 2 : 1; }
// The other pairs of an XCD are taken `group` at a time, a group's tiles by rank: all its longest tiles first,
// then all its second longest (map_group chooses).
S2_HD inline bool map_workgroup(int wg, int bh_total, int tiles, int group, int& bh, int& rank) {
  const int x = wg & 7, per_xcd = bh_total >> 3, left = bh_total & 7;
  int slot = wg >> 3;
  if (left > 0) {  // an XCD's slots for what is left over come first
    const int run = deal_run(tiles), runs = (tiles + run - 1) / run, shared = run * ((left * runs + 7) >> 3);
    if (slot < shared) {
      const int i = 8 * (slot / run) + x, r = i / left;
      rank = r * run + slot % run;
      bh = 8 * per_xcd + i - r * left;
      return rank < tiles;
    }
    slot -= shared;
  }
  const int g = slot / (group * tiles);
  if (group == 1) {
    rank = slot - g * tiles;
    bh = x + 8 * g;
    return g < per_xcd;
  }
  const int in = slot - g * (group * tiles);
  const int size = group < per_xcd - g * group ? group : per_xcd - g * group;
  if (size <= 0) return false;
  rank = in / size;
  bh = x + 8 * (g * group + in - rank * size);
  return true;
}
S2_HD inline int grid_for(int bh_total, int tiles) {
  const int left = bh_total & 7, run = deal_run(tiles), runs = (tiles + run - 1) / run;
  return 8 * ((bh_total >> 3) * tiles + run * ((left * runs + 7) >> 3));
}
// Same XCD assignment, but the (batch, head) pairs are interleaved: all their longest
// tiles are dispatched first, then all their second longest, ...  Used where tile lengths are very
// uneven (key tiles on a stripe are attended by hundreds of query blocks, the others by a few), so
// that the longest tile of the last head does not start late and become the tail of the launch.
// (Where pairs are left over the unit is the run: of run r of every pair an XCD has bh_total / 8, those of its own pairs, and one of what is
// left over if there is one among numbers r * left, r * left + 1, ... that is its own modulo 8.  That makes (r * bh_total + 7 - x) / 8
// before run r, and so the s-th run of XCD x is one of number (8 * s + x) / bh_total.  The XCD takes the tiles of its runs of one number by rank.)
S2_HD inline bool map_workgroup_interleaved(int wg, int bh_total, int tiles, int& bh, int& rank) {
  const int x = wg & 7, per_xcd = bh_total >> 3, left = bh_total & 7;
  const int run = left > 0 ? deal_run(tiles) : 1;
  const int slot = wg >> 3, r = (8 * (slot / run) + x) / bh_total;
  const unsigned upto = (unsigned)r * bh_total + 7 - x;
  const int before = upto >> 3, of_run = (int)((upto + bh_total) >> 3) - before;  // of_run: pairs of which the XCD has run r
  const int i = slot - before * run, in_run = i / of_run, in = i - in_run * of_run;
  rank = r * run + in_run;
  bh = in < per_xcd ? x + 8 * in : 8 * per_xcd + ((x - r * left) & 7);
  return rank < tiles;
}
S2_HD inline int grid_for_interleaved(int bh_total, int tiles) {
  const int run = (bh_total & 7) > 0 ? deal_run(tiles) : 1, runs = (tiles + run - 1) / run;
  return (int)(((unsigned)bh_total * runs + 7) / 8 * 8) * run;
}
// How many pairs of an XCD to take at a time.  One after the other leaves the longest tiles of the last
// pair for the end of the launch, which counts when an XCD's 64 workgroup slots go round only a few
// times: forward / dQ of 2 x 16 heads x 4096 x 64 36.1 / 46.6 us one by one, 32.9 / 42.6 in fours; dense 32
// heads x 8192 542 / 781 and 518 / 731.
// From about eight rounds on the tail is nothing, while four heads' stripes then share an L2: 32 heads x
// 32768 the same both ways, 32 heads x 131072 (2 MB of stripes a head) 5.90 ms one by one, 6.06 in fours.
// Pairs of a packed batch are of different lengths and go one after the other: neighbouring workgroups of an
// XCD go to its four shader engines in turn, so with four pairs side by side each engine had the tiles of
// one, and the launch waited for the engine with the longest sequence.  Forward / dQ of 20 x 5 heads x up to
// 8832 x 128 197.7 / 277.4 us in fours, 119.2 / 166.5 one by one; 11 x 10 heads x 64 87.7 / 107.7 and 61.2 / 76.8;
// 8 x 32 heads of 200 to 8192 rows 330.8 / 448.4 and 331.6 / 454.1.
inline int map_group(int bh_total, int tiles, bool packed) {
  return !packed && (int64_t)((bh_total + 7) / 8) * tiles <= 8 * 64 ? 4 : 1;
}

}  // namespace s2
