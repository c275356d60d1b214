// Which wave takes which entry of a list, apart from HIP so that a CPU test can compile it.
#pragma once

namespace da {
namespace ring {

// Entry number `turn` of a group's walk goes to this one of its `parts` (2, 4 or 8) waves.  sub: entries per key block.  A
// block of 128 slots is two entries in a row; the waves change places from one block to the next, else one of two waves had
// the first half of every block, and of peaked attention what matters to the first 64 queries of a block is mostly there.
// (24 heads x 990 blocks of 8x16, 99 kept, peaked 13.26 -> 12.29 ms; 5 heads, 21 frames, a quarter kept 2.96 -> 2.52 ms; nothing
// dropped the same.)
constexpr int wave_of_turn(int turn, int sub, int parts) { return (sub == 1 ? turn : turn + (turn >> 1)) & (parts - 1); }

}  // namespace ring
}  // namespace da
