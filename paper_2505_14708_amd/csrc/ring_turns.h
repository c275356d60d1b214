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

// LDS beside the ring that a workgroup of 8 / 2^split groups of 64 queries needs: the bitmaps of its query blocks (g bits each), the
// union of their lists (an entry is four bytes; sub of them to a block) and 512 bytes of the ring's state.
constexpr int AUX_BYTES = 32 * 1024;
constexpr int kValidBit = 18;                         // (key sub-blocks are numbered below 2^18; the lists take more LDS than there is long before)
inline long long aux_bytes(long long g, long long k, int sub, bool any_length, int split) {
  const long long blocks = 8 / sub >> split ? 8 / sub >> split : 1;
  const long long union_max = sub * (any_length || g < blocks * k ? g : blocks * k);
  return blocks * 4 * ((g + 31) / 32) + 4 * union_max + 512;
}
// What the kernel runs is what it ran when four groups of 64 queries were a workgroup's most: four bitmaps, and the union of four
// (sub = 2: two) lists.  Halves of a unit always fit then, whole ones up to 6451 blocks where nothing is dropped.
inline bool lists_fit(long long g, long long k, int sub, bool any_length) {
  const long long blocks = 4 / sub, union_max = sub * (any_length || g < blocks * k ? g : blocks * k);
  return g * sub < (1 << kValidBit) && 4LL * 4 * ((g + 31) / 32) + 4 * union_max + 512 <= AUX_BYTES;
}
inline int least_split(long long g, long long k, int sub, bool any_length) { return aux_bytes(g, k, sub, any_length, 0) > AUX_BYTES; }

// Either all units of a launch are shared by 2^split[0] workgroups each, and then shares without a group have none: `head_shares` to a
// head.  (A workgroup that finds nothing to do still takes a CU for 6 us, as much as all of the LDS needs to change hands: 250 heads of
// one block as eighths 21 -> 69 us if seven of eight are empty.)  Or (head_shares 0) the first `first` units are shared by 2^split[0]
// workgroups each, the others by 2^split[1].  (`first` is a multiple of eight where there are others and split[0] is not 0.)
struct Share {
  int first, split[2];
  unsigned grid;
  int head_shares;
};
// what workgroup `b` of a launch is
struct ShareOf {
  int head, unit, lsub, sub;    // share number `sub` of the 2^lsub of that unit of that head
};
// left: units of left-over frames among the per_head units of a head
DA_HOST_DEVICE inline ShareOf share_of(const Share& s, int b, int per_head, int left) {
  if (s.head_shares) {
    // (the shares of a unit are eight apart: on one XCD, but for the last few.  Where a head has only one, heads go to the XCDs in turn,
    // as in the launch that leaves K and V in their L2: 96 and 128 heads of one block 20.7 and 21.5 -> 19.8 and 20.0 us.)
    const int lsub = s.split[0], mask = (1 << lsub) - 1, stretch = b & ~(8 * mask + 7);
    const bool apart = s.head_shares > 1 && stretch + 8 * mask + 8 <= (int)s.grid;
    const int nth = apart ? stretch + ((b & 7) << lsub) + ((b >> 3) & mask) : b;
    const int head = nth / s.head_shares, r = nth - head * s.head_shares;
    // (the last unit of left-over frames, the one with empty places, is a head's last one here)
    const int unit = (r >> lsub) + left;
    return {head, unit < per_head ? unit : unit - per_head, lsub, r & mask};
  }
  const int past = b - (s.first << s.split[0]);
  const int lsub = past < 0 ? s.split[0] : s.split[1], nth = past < 0 ? b : past;
  // (the shares of a unit are eight apart: on one XCD)
  const int unit = (past < 0 ? 0 : s.first) + (nth >> (3 + lsub)) * 8 + (nth & 7), head = unit / per_head;
  return {head, unit - head * per_head, lsub, (nth >> 3) & ((1 << lsub) - 1)};
}

// A workgroup fills a CU, so a launch of few comes in rounds of kCUs and the last round takes as long as a full one
// however few are in it.  With two, four or eight workgroups to a unit there are as many times the waves to each list, and a
// workgroup is done in about 0.55, 0.35 and 0.25 of the time (tiles are shared by fewer, the fixed part stays).  Times of
// da_forward in us, whole units / halves / quarters / eighths (bold what is taken; units of a list of k entries each):
//   - as many shares as fit in one round: 18 units of 24 tiles 64 / 46 / 41 / *38*,
//     26 of 52 174 / 120 / 97 / *82*, 36 of 17 129 / 106 / *95* / 108, 45 of 7 75 / 59 / *56* / 71, 90 of 12 104 / *81* / 89, 120 of 96 360 /
//     *234* / 267.  With the empty shares launched as well these were too many for a round: 36 heads of 28 blocks, 252 halves, 14
//     kept 94 -> 76, 12 heads of 84, 42 kept 149 -> 119, 6 heads 105 -> 80 (quarters), 9 heads of 28, 14 kept 54 -> 49 (eighths);
//   - up to three quarters of a round, as halves but for 64 as quarters, so that a CU has two at most (whole / *so*): 136 of 40 176 / *171*, 152 of 30 130 / *118*, 160 of 64 248 / *240*, 192 of 120 428 / *416*; lists of any length, whatever their average: 132 of 26
//     232 / *167*, 165 of 6 165 / *130*, 168 of 17 368 / *246*, 180 of 29 220 / *185*.  Not where all lists are short, for the fixed part is most of it
//     (144 of 8 *84* / 86, 160 of 3 *63* / 69, 171 of 18 *115* / 119, 180 of 9 *94* / 97; 156 of 16 *104* / 102), nor where a CU would get three
//     (189 of 42 *192* / 230, 190 of 75 *312* / 364).  More units are whole: 208 of 64 *270* / 326, 240 of 28 *169* / 202;
//   - up to four rounds, what a last round has of at most half: up to 64 units as quarters (288 of 64 499 / *371*, 576 of 64 785 /
//     *674*), more as halves (384 of 64 516 / *456*, 896 of 64 1080 / *1033*, 640 of 64 799 / *737*).  Up to three quarters of a round, 64 as
//     quarters, for units seldom last as long as one another (396 of 14 235 / *207*, 648 of 65 573 / *528*, 656 of 81 605 / *557*, 960 of
//     256 2154 / *1998*, 414 of 9 169 / *161*; on 32 others from 4 % worse to 5 % better, 0.4 % better on average).  A fuller or full one
//     stays (504 of 570 *4069* / 4510, of 65 *614* / 661, 750 of 300 *2026* / 2093; units that do last as long: 512 of 64 *589* / 639, 768 *878* / 923, 1024
//     *1174* / 1223, but 448 541 / *548*).  Lists of any length, whose units end at different times: 64 as quarters (1024 of 102 on average
//     2278 / *2110*), and in the second half of the second round all others as halves (64 as quarters / *so*: 408 of 56 455 / *391*, 418 of 88
//     694 / *623*, 450 of 240 1457 / *1312*, 500 of 200 1716 / *1466*, 504 of 52 413 / *421*; not short ones, 420 of 14 *247* / 254.  Towards the end of
//     that range it depends on how peaked they are: 456 of 96 peaked 504 / *518*, 480 of 101 586 / *613*, 504 of 144 696 / *726*, but with q
//     scaled by 1/4 432 of 96 572 / *552*, 480 670 / *640*, 512 of 204 1886 / *1883*; up to 450, peaked or not, 2 to 8 % are gained);
//   - and 64 as halves after that, for units differ in length: 5952 of 198 12080, *11918*, nothing dropped 20167, *20103*.
constexpr int kCUs = 256;
constexpr int kShortList = 24;
// head_groups: groups of 64 queries of a head; tiles: entries of a list (on average, where they are of any length); least: units are
// shared by at least 2^least (LDS)
inline Share share_out(long long heads, long long head_groups, long long tiles, bool any_length, int least) {
  const long long total = heads * ((head_groups + 7) / 8);
  if (least == 0 && head_groups <= 4) least = 1;      // (whole units would be half empty, with nothing for the waves of that half to do)
  int all = 3;
  while (all > least && heads * ((head_groups + (8 >> all) - 1) / (8 >> all)) > kCUs) --all;
  if (all) {
    const int head_shares = (int)((head_groups + (8 >> all) - 1) / (8 >> all));
    return {0, {all, all}, (unsigned)(heads * head_shares), head_shares};
  }
  int split[2] = {0, 0};                              // (more than kCUs halves, hence more than kCUs / 2 units, from here on)
  long long rest = 0;
  if (total <= kCUs / 4 * 3) {
    // (beyond 184 units rounding up to eights leaves a third share to some CU unless there is nothing to round)
    if ((total % 8 == 0 || total < kCUs / 4 * 3 - 8) && (any_length || tiles >= kShortList)) split[0] = 1, split[1] = 2, rest = kCUs / 4;
  } else if (total > kCUs && total <= 4 * kCUs) {
    const int last = (int)(total % kCUs);
    if (any_length && total > kCUs / 2 * 3 && total <= 2 * kCUs && tiles >= kShortList) split[0] = 1, split[1] = 2, rest = kCUs / 4;
    else if (last > kCUs / 4 && last <= kCUs / 2) split[1] = 1, rest = last;
    else if (any_length || (last > 0 && last <= kCUs / 4 * 3)) split[1] = 2, rest = kCUs / 4;
  } else if (total > kCUs) split[1] = 1, rest = kCUs / 4;
  if (rest >= total) rest = 0;
  if (rest && split[0]) rest += (total - rest) % 8;
  Share s = {(int)(rest ? total - rest : (total + 7) / 8 * 8), {split[0], split[1]}, 0, 0};
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
