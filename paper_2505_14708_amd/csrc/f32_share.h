// How the float32 attention deals its work out, apart from HIP so that a CPU test can compile it.
#pragma once

#ifdef __HIPCC__
#define DA_F32_HOST_DEVICE __host__ __device__
#else
#define DA_F32_HOST_DEVICE
#endif

namespace da {

// Half query blocks (32 queries) come in eight stretches of `chunk`, one per XCD (workgroups are dealt round-robin to them, and
// consecutive blocks have much of their lists in common).  The first `whole` of a stretch are a workgroup each, the
// others are two workgroups of 16 queries.
struct F32Share {
  long long chunk, whole;
  unsigned grid;
};
struct F32Piece {
  long long half;         // number of the half block (the last stretch may have fewer than `chunk`: then past the end)
  int second, queries;    // its second 16 queries; 32 or 16
};
DA_F32_HOST_DEVICE inline F32Piece f32_piece(const F32Share& s, unsigned b) {
  const long long at = b >> 3, past = at - s.whole;
  if (past < 0) return {(b & 7) * s.chunk + at, 0, 32};
  return {(b & 7) * s.chunk + s.whole + (past >> 1), (int)(past & 1), 16};
}

// A half block is one workgroup of four waves; `places` of them run at a time on an XCD's 32 CUs.  Two pieces of 16 queries read
// K and V twice, so a launch of nothing else loses (H x blocks, da_forward in us, halves / *taken*):
//   - where there is a CU for every piece, all: 2 x 8 (64 channels) 21.6 / *18.1*, 1 x 28 38.3 / *29.6*; with 64 channels up to
//     two to a CU: 4 x 28 29.0 / *28.3*, 2 x 60 41.4 / *40.4* (128 channels, pieces / halves: 4 x 28 40.2 / *39.2*, 2 x 56 60.0 / *58.6*);
//   - else the last, partial round of halves where it is short, so that its waves find others to share a SIMD with and
//     are done in half the time.  `even`: every half block holds a valid query, and lists are of one length.  Then that
//     is at most half as many halves as CUs (a CU gets one piece instead of one half or none), or with 128 channels a few
//     more than CUs (some would get two halves); four heads, c halves to an XCD, 30 % kept: 128 channels, 64 places: 68
//     179 / *155*, 80 202 / *177*, 84 *217* / 220 in pieces, 91 *233* / 237, 96 *240* / 245, 100 313 / *290*, 104 332 /
//     *308*, 168 747 / *706*, 232 1336 / *1281*; 64 channels, 96 places: 100 183 / *163*, 112 204 / *182*, 116 *209* /
//     211, 204 583 / *543*, 212 *600* / 605.  Else the round's workgroups do not all last as long and the line need not
//     be drawn there: lists of any length, 1 x 840 (18 halves in the last round) 1630 / *1549*; some halves without a
//     query, 4 x 84 191 / *164*, 5 x 112 332 / *309*, 8 x 84 297 / *286*, 12 x 112 689 / *675*, 12 x 140 1046 / *1027*
//     (30x52 frames; last rounds of 17 to 32 halves on 19 other grids: 7 to 16 % gained on seven, 2 to 5 on seven,
//     nothing on four, 2.6 lost on one, and 2.5 on 7 x 125 of 33x33 with all kept), 16 x 28 (64 channels) 92 / *85*, but
//     6 x 84 (62 of 64 places) *225* / 230, and with 64 channels 8 x 112 (32 of 96) *262* / 267.
inline F32Share f32_share_out(long long halves, bool even, int d) {
  const long long cus = 32, places = d == 64 ? 3 * cus : 2 * cus;   // (registers)
  const long long all = d == 64 ? cus : cus / 2, short_round = d == 64 ? 20 : 40;
  F32Share s;
  s.chunk = (halves + 7) / 8;
  const long long last = s.chunk % places;
  const bool is_short = last <= short_round && !(even && last > cus / 2 && last <= cus);
  s.whole = s.chunk <= all ? 0 : s.chunk > places && is_short ? s.chunk - last : s.chunk;
  s.grid = (unsigned)(8 * (s.whole + 2 * (s.chunk - s.whole)));
  return s;
}

}  // namespace da
