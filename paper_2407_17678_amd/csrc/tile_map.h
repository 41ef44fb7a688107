// Internal: which tile a workgroup computes.  (Plain arithmetic, so that a test can go through it on the host.)
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#define S2_HD __host__ __device__
#else
#define S2_HD
#endif

namespace s2 {

// n / d of 0 <= n < 2^31 for a d that the host knows: n * ceil(2^(31 + l) / d) >> (31 + l), 2^l the first power of two from d on (Granlund
// and Montgomery's division by invariant integers).  Rounding the factor up adds less than 2^l / 2^(31 + l) / d * n < 1 / d to the
// quotient, which does not reach the next whole number.  Three scalar instructions; the division that the compiler writes goes
// through a vector reciprocal and back, and a tile's start had five to seven of them.  With them gone and a tile's record in one
// scalar load (DevTiles in kernels.h), forward and backward, us: packed 13 x 18 heads of 100 to 6272 rows x 64 54.6 -> 51.5, 168 -> 162, 20 x 11 heads x 128
// 146 -> 139, 423 -> 410, 8 x 32 heads 326 -> 323, 974 -> 961; 1 x 4 x 512 x 64 8.3 -> 7.9, 15.8 -> 15.7; 2 x 16 x 3904 x 128 45.5 -> 45.0, 129.4 -> 128.8.
struct FastDiv {
  uint32_t factor, shift;
};
inline FastDiv fast_div(uint32_t d) {
  FastDiv f{0, 31};
  while (((uint64_t)1 << (f.shift - 31)) < d) ++f.shift;
  f.factor = (uint32_t)((((uint64_t)1 << f.shift) + d - 1) / d);
  return f;
}
S2_HD inline int operator/(int n, const FastDiv& f) { return (int)(((uint64_t)(uint32_t)n * f.factor) >> f.shift); }

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
// Over 947 launches of drawn cases 10 % faster in the mean than an XCD to a pair and 2.5 % slower at worst; over 246 of packed batches 3 % faster in the mean.  Where an XCD to a pair
// is known to be ahead: dense backward 1 x 25 heads x 1280 x 128 56.0 and 58.5 (31 or 32 key tiles to an XCD, so that its longest query tiles go to the compute units of its longest
// key tiles), dS kept 2 x 31 x 1152 92.6 and 96.8, 1 x 23 x 992 in blocks of 16 37.3 and 38.4; packed, where it depends on whose pairs are left over, forward 3 x 6 heads of up to
// 6528 rows x 64 29.0 and 33.6, 2 x 39 in blocks of 32 85.8 and 89.2, backward 15 x 15 in blocks of 16 834 and 911, 20 x 5 770 and 805, 11 x 6 561 and 581.
inline int deal_run_shift(int tiles) { return tiles >= 128 ? 2 : tiles >= 64 ? 1 : 0; }
// The pairs interleaved: all their longest
// tiles are dispatched first, then all their second longest, ...  Used where tile lengths are very
// uneven (key tiles on a stripe are attended by hundreds of query blocks, the others by a few), so
// that the longest tile of the last head does not start late and become the tail of the launch.
// (Where pairs are left over the unit is the run: of run r of every pair an XCD has bh_total / 8, those of its own pairs, and one of what is
// left over if there is one among numbers r * left, r * left + 1, ... that is its own modulo 8.  That makes (r * bh_total + 7 - x) / 8
// before run r, and so the s-th run of XCD x is one of number (8 * s + x) / bh_total.  The XCD takes the tiles of its runs of one number by rank.)
struct KeyMap {
  int bh_total, tiles, run;                   // run: shift of the tiles to a run
  FastDiv by_total, by_own, by_more;          // division by bh_total, bh_total / 8 and bh_total / 8 + 1
  // (of whole runs, so up to a run less one more to a pair than it has tiles)
  int64_t grid() const { return ((int64_t)bh_total * ((tiles + (1 << run) - 1) >> run) + 7) / 8 * 8 << run; }
};
inline KeyMap key_map(int bh_total, int tiles) {
  KeyMap m{};
  m.bh_total = bh_total;
  m.tiles = tiles;
  m.run = (bh_total & 7) > 0 ? deal_run_shift(tiles) : 0;
  m.by_total = fast_div(bh_total);
  m.by_own = fast_div(bh_total >= 8 ? bh_total >> 3 : 1);
  m.by_more = fast_div((bh_total >> 3) + 1);
  return m;
}
S2_HD inline bool map_workgroup_interleaved(const KeyMap& m, int wg, int& bh, int& rank) {
  const int x = wg & 7, per_xcd = m.bh_total >> 3, left = m.bh_total & 7;
  const int slot = wg >> 3, r = (8 * (slot >> m.run) + x) / m.by_total;
  const unsigned upto = (unsigned)r * m.bh_total + 7 - x;
  const int before = upto >> 3, of_run = (int)((upto + m.bh_total) >> 3) - before;  // of_run: pairs of which the XCD has run r
  const int i = slot - (before << m.run), in_run = of_run > per_xcd ? i / m.by_more : i / m.by_own, in = i - in_run * of_run;
  rank = (r << m.run) + in_run;
  bh = in < per_xcd ? x + 8 * in : 8 * per_xcd + ((x - r * left) & 7);
  return rank < m.tiles;
}
// Row tiles.  The own pairs of an XCD are taken a group of one or four at a time, a group's tiles by rank: all its longest tiles first,
// then all its second longest (map_group chooses).  What is left over comes first, by itself; or last, interleaved with the last `dealt` of
// the own pairs (dealt_pairs chooses).
struct RowMap {
  int per_xcd, left;    // pairs of an XCD's own, and left over
  int tiles;            // of a pair
  int run, shared;      // shift of the tiles to a run; an XCD's slots for what is left over where that comes first
  int plain, before;    // an XCD's slots for the pairs taken in groups; so many pairs are before those that are interleaved
  KeyMap dealt;         // the interleaved ones
  int group, in_group;  // shift of the pairs to a group, tiles of a group
  FastDiv by_left, by_group, by_last;  // division by left, in_group and the pairs of the last group
  int64_t grid() const { return 8 * ((int64_t)plain + shared) + dealt.grid(); }
};
// How many of an XCD's own pairs are interleaved with what is left over; -1: that comes first.
// First means that its short tiles, too, run before the longest of the own pairs, which a launch of few rounds of the chip's workgroup
// slots cannot make up for.  So whole sequences interleave all pairs, up to four rounds where an XCD has more than one group of four,
// and where five or more are left over up to one, or one and a half of dense tiles, whose lengths differ most.  Forward, us, first and interleaved: dense
// 2 x 25 heads x 3072 x 64 103 and 81, 1 x 39 x 2048 x 64 39.9 and 37.4, 2 x 27 x 2048 x 128 82 and 71, 1 x 14 x 5504 141 and 117, sparse 1 x 15 x 4096 x 128 28.3
// and 26.0, 4 x 21 x 512 17.8 and 15.3, but 1 x 23 x 3136 (1.1 rounds) 25.5 and 27.9; backward, dense 3 x 26 x 640 x 128 54.0 and 45.0, sparse 1 x 31 x 512
// 27.2 and 25.4.  With one group and fewer left over neither wins (forward of 131 cases 0.94 to 1.08 of the other, 1.00 in the mean); with more
// rounds the pairs push each other's stripes out of the L2s (4 x 37 heads x 3200 x 128, blocks of 128, 168 and 175).
// Rows against a cache are tiles of one length, and only their L2 matters: the last group and what is left over are interleaved
// after the other groups.  First, all interleaved and so: 3 x 23 heads, 1152 rows against 51072 351, 345 and 335; 4 x 37, 1024 against 16896 196, 208 and 195; 3 x 7, 3584
// against 48256 152, 142 and 142.
enum RowTiles { kRowsOfCache, kSparseRows, kDenseRows };  // of some rows against a cache; of whole sequences
inline int dealt_pairs(int bh_total, int tiles, int group, RowTiles of, int slots) {
  const int own = bh_total >> 3, left = bh_total & 7;
  if (left == 0 || group != 4) return -1;
  if (of == kRowsOfCache) return own > 0 ? (own - 1) % 4 + 1 : 0;
  const int64_t halves = own > 4 ? 8 : left < 5 ? 0 : of == kDenseRows ? 3 : 2;  // half rounds
  return (int64_t)bh_total * tiles <= halves * 4 * slots ? own : -1;
}
// Workgroups of the row-tile kernels that an XCD's 32 compute units hold.
inline int xcd_slots(int head_dim) { return head_dim == 128 ? 64 : 96; }
inline RowMap row_map(int bh_total, int tiles, int group, RowTiles of, int slots) {
  RowMap m{};
  m.per_xcd = bh_total >> 3;
  m.left = bh_total & 7;
  m.tiles = tiles;
  m.run = deal_run_shift(tiles);
  const int dealt = dealt_pairs(bh_total, tiles, group, of, slots);
  if (dealt < 0) {
    m.shared = ((m.left * ((tiles + (1 << m.run) - 1) >> m.run) + 7) >> 3) << m.run;
    m.plain = m.per_xcd * tiles;
  } else {
    m.plain = (m.per_xcd - dealt) * tiles;
    m.before = 8 * (m.per_xcd - dealt);
    m.dealt = key_map(8 * dealt + m.left, tiles);
  }
  m.group = group == 4 ? 2 : 0;
  m.in_group = tiles << m.group;
  m.by_left = fast_div(m.left > 0 ? m.left : 1);
  m.by_group = fast_div(m.in_group);
  const int last = m.per_xcd & ((1 << m.group) - 1);
  m.by_last = fast_div(last > 0 ? last : 1);
  return m;
}
S2_HD inline bool map_workgroup(const RowMap& m, int wg, int& bh, int& rank) {
#ifdef __HIP_DEVICE_COMPILE__
  // All of it is loaded at once: left alone, each branch asks for its part of the arguments and waits (forward of 1 x 4 heads x 512 x 64 7.9 -> 8.2 us).
  asm volatile("" ::"s"(m.per_xcd), "s"(m.left), "s"(m.tiles), "s"(m.run), "s"(m.shared), "s"(m.plain), "s"(m.before), "s"(m.group), "s"(m.in_group),
               "s"(m.by_left.factor), "s"(m.by_left.shift), "s"(m.by_group.factor), "s"(m.by_group.shift), "s"(m.by_last.factor), "s"(m.by_last.shift),
               "s"(m.dealt.bh_total), "s"(m.dealt.tiles), "s"(m.dealt.run), "s"(m.dealt.by_total.factor), "s"(m.dealt.by_total.shift),
               "s"(m.dealt.by_own.factor), "s"(m.dealt.by_own.shift), "s"(m.dealt.by_more.factor), "s"(m.dealt.by_more.shift));
#endif
  const int x = wg & 7;
  int slot = wg >> 3;
  if (slot < m.shared) {
    const int i = 8 * (slot >> m.run) + x, r = i / m.by_left;
    rank = (r << m.run) + (slot & ((1 << m.run) - 1));
    bh = 8 * m.per_xcd + i - r * m.left;
    return rank < m.tiles;
  }
  slot -= m.shared;
  if (slot >= m.plain) {
    const bool any = map_workgroup_interleaved(m.dealt, 8 * (slot - m.plain) + x, bh, rank);
    bh += m.before;
    return any;
  }
  const int g = slot / m.by_group, in = slot - g * m.in_group;
  const int size = m.per_xcd - (g << m.group);  // pairs from the group on
  int of_rank;
  if (size >> m.group) {
    rank = in >> m.group;
    of_rank = in & ((1 << m.group) - 1);
  } else {
    rank = in / m.by_last;
    of_rank = in - rank * size;
  }
  bh = x + 8 * ((g << m.group) + of_rank);
  return size > 0;
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
