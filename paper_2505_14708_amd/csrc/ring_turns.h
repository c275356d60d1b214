// How the bf16 attention deals its work out, apart from HIP so that a CPU test can compile it: units of eight groups of 64
// queries, how many workgroups share a unit, which of the waves that share a list takes which entry of it, and the key that orders a walk.
#pragma once

#ifdef __HIPCC__
#define DA_HOST_DEVICE __host__ __device__
#else
#define DA_HOST_DEVICE
#endif

namespace da {
namespace ring {

// A head's query blocks, `fg` (a power of two) to a unit: fg consecutive frames of one position where there are that many.  The
// frames left over at the end are put end to end, position after position, and that row is cut into units (their lists
// have less in common: they come first).  A position's left-over frames then lie in one unit or in two next to each other, and only the
// head's last such unit has empty places.
// (Taken four, two and one frames at a time, of as many positions as fill a unit, three frames of a position lie in two units among
// blocks of other positions.  da_forward, us, 24 heads of 45x80, 10 % kept: 3 frames 309 -> 287, 7 1168 -> 1091, 15 4631 -> 4490, 31 17882 -> 17579; 8
// heads of 30x52, a quarter kept: 3 frames 84.5 -> 79.8, 7 227 -> 212, 15 801 -> 776, but 5 151.9 -> 154.5.)
struct UnitPlace {
  int pos0, first, frames, frame0;   // block w of the unit is number `first` + w of a row that is `frames` frames of pos0, then of pos0 + 1, ...
  int recip;                         // 256 / frames, rounded up: divides numbers below 16 exactly
};
DA_HOST_DEVICE inline int left_units(int T, int fg, int per_frame) { return (per_frame * (T & (fg - 1)) + fg - 1) / fg; }
DA_HOST_DEVICE inline int units_per_head(int T, int fg, int per_frame) { return T / fg * per_frame + left_units(T, fg, per_frame); }
// unit number n of a head
DA_HOST_DEVICE inline UnitPlace unit_place(int n, int T, int log_fg, int per_frame) {
  const int fg = 1 << log_fg, left = T & (fg - 1), past = n - left_units(T, fg, per_frame);
  if (past < 0) {
    const int pos0 = (n << log_fg) / left;
    return {pos0, (n << log_fg) - pos0 * left, left, T - left, (255 + left) / left};
  }
  const int groups = T >> log_fg, pos0 = past / groups;
  return {pos0, 0, fg, (past - pos0 * groups) << log_fg, 256 >> log_fg};
}
// the position and the frame of its block w (the position may lie past the last one: an empty place, and so are all after it)
DA_HOST_DEVICE inline int unit_pos(const UnitPlace& u, int w) { return u.pos0 + (((u.first + w) * u.recip) >> 8); }
DA_HOST_DEVICE inline int unit_frame(const UnitPlace& u, int w) { return u.frame0 + u.first + w - (((u.first + w) * u.recip) >> 8) * u.frames; }

// The first `first` units of a launch are shared by 2^split[0] workgroups each, the others by 2^split[1].  (`first` is a
// multiple of eight where there are others and split[0] is not 0.)
struct Share {
  int first, split[2];
  unsigned grid;
};
// what workgroup `b` of a launch is
struct ShareOf {
  int unit, lsub, sub;    // share number `sub` of the 2^lsub of that unit
};
DA_HOST_DEVICE inline ShareOf share_of(const Share& s, int b) {
  const int past = b - (s.first << s.split[0]);
  const int lsub = past < 0 ? s.split[0] : s.split[1], nth = past < 0 ? b : past;
  // (the shares of a unit are eight apart: on one XCD)
  return {(past < 0 ? 0 : s.first) + (nth >> (3 + lsub)) * 8 + (nth & 7), lsub, (nth >> 3) & ((1 << lsub) - 1)};
}

// A workgroup fills a CU, so a launch of few comes in rounds of kCUs and the last round takes as long as a full one
// however few are in it.  With two, four or eight workgroups to a unit there are as many times the waves to each list, and a
// workgroup is done in about 0.55, 0.35 and 0.25 of the time (tiles are shared by fewer, the fixed part stays).  Times of
// da_forward in us, whole units / halves / quarters / eighths (bold what is taken; units of a list of k entries each):
//   - at most half a round is shared out so that it fills one: 18 units of 24 tiles 64 / 46 / 41 / *38*, 26 of 52 174 / 120 /
//     97 / *82*, 36 of 17 129 / 106 / *95* / 108, 45 of 7 75 / 59 / *56* / 71, 90 of 12 104 / *81* / 89, 120 of 96 360 / *234* / 267;
//   - up to three quarters of a round, as halves but for 64 as quarters, so that a CU has two at most (whole / *so*): 136 of 40 176 / 171, of 120 397 /
//     370, 160 of 64 248 / 240, 176 of 64 254 / 246, 192 of 120 428 / 416.  Not where lists are short, for the fixed part is most of it
//     (144 of 20 *121* / 123, 176 of 28 *148* / 151, 192 of 28 *152* / 158), nor where a CU would get three (189 of 42 *192* / 230, 190 of
//     75 *312* / 364).  More units are whole: 208 of 64 *270* / 326, 240 of 28 *169* / 202;
//   - up to four rounds, what a last round has of at most half: up to 64 units as quarters (288 of 64 499 / 371, 576 of 64 785 /
//     674), more as halves (384 of 64 516 / 456, 896 of 64 1080 / 1033; 640 of 64 799 / 737).  A fuller or full one stays (512 of 64 *589* / 639 with 64 as quarters,
//     768 *878* / 923, 1024 *1174* / 1223, 448 *541* / 548), but for lists of any length, whose units end at different times: 1024 of
//     102 on average 2278 / *2110*;
//   - and 64 as halves after that, for units differ in length: 5952 of 198 12080, *11918*, nothing dropped 20167, *20103*.
constexpr int kCUs = 256;
constexpr int kLongList = 36;
// total: units of the launch; tiles: entries of a list (on average, where they are of any length); least: units are shared by at
// least 2^least (LDS)
inline Share share_out(long long total, long long tiles, bool any_length, int least) {
  int split[2] = {0, 0};
  long long rest = 0;
  if (total <= kCUs / 8) split[0] = 3;
  else if (total <= kCUs / 4) split[0] = 2;
  else if (total <= kCUs / 2) split[0] = 1;
  else if (total <= kCUs / 4 * 3 && (total % 8 == 0 || total < kCUs / 4 * 3 - 8) && tiles >= kLongList) split[0] = 1, split[1] = 2, rest = kCUs / 4;
  else if (total > kCUs && total <= 4 * kCUs) {
    const int last = (int)(total % kCUs);
    if (last > kCUs / 4 && last <= kCUs / 2) split[1] = 1, rest = last;
    else if (any_length || (last > 0 && last <= kCUs / 4)) split[1] = 2, rest = kCUs / 4;
  } else if (total > kCUs) split[1] = 1, rest = kCUs / 4;
  for (int& x : split) x = x < least ? least : x;
  if (rest && split[0]) rest += (total - rest) % 8;
  Share s = {(int)(rest ? total - rest : (total + 7) / 8 * 8), {split[0], split[1]}, 0};
  s.grid = ((unsigned)s.first << split[0]) + ((unsigned)((rest + 7) / 8 * 8) << split[1]);
  return s;
}

// Entry number `turn` of a group's walk goes to this one of its `parts` (1, 2, 4 or 8) waves.  sub: entries per key block.  A
// block of 128 slots is two entries in a row; the waves change places from one block to the next, else one of two waves had
// the first half of every block, and of peaked attention what matters to the first 64 queries of a block is mostly there.
// (24 heads x 990 blocks of 8x16, 99 kept, peaked, two waves to a list 13.26 -> 12.29 ms; 5 heads, 21 frames, a quarter kept
// 2.96 -> 2.52 ms; nothing dropped the same.)
DA_HOST_DEVICE constexpr int wave_of_turn(int turn, int sub, int parts) { return (sub == 1 ? turn : turn + (turn >> 1)) & (parts - 1); }

// The order of a walk: entry number p of a class of 1 / inv_total entries goes by the key (p + u) / (number of entries), u the
// fraction of the class's number times the golden section; the sort puts keys (below 1 but for rounding) into buckets first.
constexpr int kWalkBuckets = 2048;
DA_HOST_DEVICE inline float walk_key(int cls, int p, float inv_total) {
  const float u = (float)cls * 0.618034f;
  return ((float)p + (u - (float)(int)u)) * inv_total;
}
DA_HOST_DEVICE inline int walk_bucket(float key) {
  const int b = (int)(key * (float)kWalkBuckets);
  return b < kWalkBuckets - 1 ? b : kWalkBuckets - 1;
}

}  // namespace ring
}  // namespace da
