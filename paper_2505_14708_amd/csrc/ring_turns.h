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

// A head's query blocks, `fg` (a power of two) to a unit: fg consecutive frames of one position where there are that many, and
// of the frames left over a power of two at a time (4, 2, 1), the same frames of fg / 4, fg / 2, fg positions together.
// (Position by position those would leave most of a unit's places empty.)  The units of the left-over frames, whose lists
// have less in common, come first, the fewest frames before the others; then a position's groups of frames one after the other.
struct UnitPlace {
  int pos0, frame0, lg;   // query block w of the unit is position pos0 + (w >> lg), frame frame0 + w mod 2^lg
};
DA_HOST_DEVICE inline int left_units(int nf, int left, int fg, int per_frame) { return left & nf ? (per_frame * nf + fg - 1) / fg : 0; }
DA_HOST_DEVICE inline int all_left_units(int T, int fg, int per_frame) {
  int n = 0;
  for (int nf = 1; nf < fg; nf <<= 1) n += left_units(nf, T & (fg - 1), fg, per_frame);
  return n;
}
DA_HOST_DEVICE inline int units_per_head(int T, int fg, int per_frame) {
  return T / fg * per_frame + all_left_units(T, fg, per_frame);
}
// unit number n of a head
DA_HOST_DEVICE inline UnitPlace unit_place(int n, int T, int log_fg, int per_frame) {
  const int fg = 1 << log_fg, left = T & (fg - 1);
  UnitPlace u;
  for (u.lg = 0; u.lg < log_fg; ++u.lg) {
    const int here = left_units(1 << u.lg, left, fg, per_frame);
    if (n < here) {
      u.pos0 = n << (log_fg - u.lg);
      u.frame0 = T & ~((2 << u.lg) - 1);
      return u;
    }
    n -= here;
  }
  const int groups = T >> log_fg;
  u.pos0 = n / groups;
  u.frame0 = (n - u.pos0 * groups) << log_fg;
  return u;
}

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

// A workgroup fills a CU, so a launch of few comes in rounds of kCUs and the last round takes as long as a full one however
// few are in it.  With two, four or eight workgroups to a unit there are as many times the waves to each list, and a
// workgroup is done in about 0.55, 0.35 and 0.25 of the time (tiles are shared by fewer, the fixed part stays).  Times of
// da_forward in us, whole units / halves / quarters / eighths (bold what is taken):
//   - at most half a round is shared out so that it fills one: 18 units of 24 tiles 64 / 46 / 41 / *38*, 26 of 52 174 / 120 /
//     97 / *82*, 36 of 17 129 / 106 / *95* / 108, 45 of 7 75 / 59 / *56* / 71, 90 of 12 104 / *81* / 89, 120 of 96 360 / *234* / 267;
//   - up to three quarters of a round, as halves but for 64 as quarters (whole / *so*): 144 of 28 111 / 112, 160 of 51 253 /
//     *211*, 180 of 238 785 / *717*, 184 of 37 220 / *196*, but 144 of 14 *100* / 107, 176 of 15 *122* / 128: where lists are
//     short, the fixed part is most of it.  216 of 28 *174* / 190;
//   - up to four rounds, the last few: 288 of 58 410, 64 of them as quarters *327*; 790 of 315 4956, *4353*; 1024 lists of any length
//     (102 on average) 2278, *2110*; 360 dense ones of 720 2268, 104 of them as halves *1808*;
//   - and 64 as halves after that, for units differ in length: 5952 of 198 12080, *11918*, nothing dropped 20167, *20103*.
constexpr int kCUs = 256;
constexpr int kShortList = 24;
// total: units of the launch; tiles: entries of a list; least: units are shared by at least 2^least (LDS)
inline Share share_out(long long total, long long tiles, int least) {
  int split[2] = {0, 0};
  long long rest = 0;
  if (total <= kCUs / 8) split[0] = 3;
  else if (total <= kCUs / 4) split[0] = 2;
  else if (total <= kCUs / 2) split[0] = 1;
  else if (total <= kCUs / 4 * 3 && tiles >= kShortList) split[0] = 1, split[1] = 2, rest = kCUs / 4;
  else if (total > kCUs && total <= 4 * kCUs) {
    const int last = (int)(total % kCUs);
    if (last > kCUs / 4 && last <= kCUs / 2) split[1] = 1, rest = last;
    else split[1] = 2, rest = kCUs / 4;
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
