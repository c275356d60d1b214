// SparseAttn for bf16 storage, d = 128, blocks of 64 or 128 tokens, on the CDNA4 matrix cores
// (v_mfma_f32_32x32x16_bf16, float32 accumulation): the shared-ring kernel.  (Described for
// 64-token blocks; what changes for 128 is said at the kernel.)
//
// Why tiles are shared.  With 64 queries against a 64-key tile the arithmetic intensity is
// 64 flop per byte of K/V, far below the machine balance, and a kernel in which every query
// block streams its own tiles is bound by the memory fabric.  Query blocks at the same patch
// position in consecutive frames keep largely the same key blocks, so a workgroup takes eight
// such blocks and walks the UNION of their lists once: every K tile of the union is brought
// into LDS once for all eight, and the V tiles they fetch meet in L2.
//
// Workgroup = 8 wavefronts, two per SIMD: while one is in its softmax (vector ALU) the other keeps the matrix pipe
// busy, and the pairing hides LDS latency, the wait for V and the waits of the ring protocol.  A wavefront owns 64
// queries (a block) and all of its list.  (Launches of few workgroups share them out among two, four or eight, with as many
// waves to a block, which take its entries in turn and put their sums together at the end: share_out.)  With four blocks to a
// workgroup and two waves to a block, as the halves of a shared one still are, the union of four lists was 1.48 lists long
// and that of eight is 2.1, so a wave's tile cost 1.4 times the bytes; there was twice the fixed part per query, and the sums of two
// waves to join.  24 heads x 1980 blocks, 198 kept: 13.4 -> 12.4 ms peaked, 21.7 -> 20.5 ms where nothing is dropped; dense, 3
// heads x 588 blocks 1.91 -> 1.74 ms.
// 64 queries are 128 registers of output, 64 of Q and 32 of scores, which leaves 32 for everything else at two
// waves per SIMD: tiles are taken 32 keys at a time, operands arrive just ahead of their use, and what can be made anew in
// the loop is not kept (opaque_lane).
//
// Per 32 keys a wave computes
//     S^T = K Q^T      (32 keys x 64 queries: 2 MFMA tiles of 32x32, 8 k-steps over d)
//     online softmax over the 32 keys
//     O^T += V^T P^T   (128 channels x 64 queries: 8 MFMA tiles, 2 k-steps over the keys)
// The transposed forms put the query on the lane axis (lane l holds query l%32), so row max and
// row sum run down a lane's own registers plus one exchange between lanes l and l^32.  Lane l
// feeds K row sigma(l%32) (sigma swaps bits 2 and 3): then the scores a lane holds in
// accumulator registers 8t..8t+7 belong to keys 16t + 8*(l/32) + 0..7 of the 32, exactly the eight
// contraction elements the P^T operand of the second product needs, so P goes from accumulator
// to operand without leaving the lane.  V arrives from the reorder step transposed and cut into
// these operands (one product step's 64 operands are one contiguous KB), so K rows are read from
// LDS, and V^T operands from global memory, as plain 16-byte pieces.
//
// The ring.  Eight 16 KB slots, each one K tile.  Tiles travel HBM/L2 -> LDS by 16-byte
// direct-to-LDS loads; the lane that writes LDS position p of row r fetches global chunk
// p ^ swizzle(r), which makes the operand reads conflict-free.  There are no workgroup barriers
// in the tile loop:
//   ready[s]   union entry whose K tile slot s holds (set once the tile has landed)
//   left[s]    how many waves have yet to read the tile in slot s (set when the tile is asked for: one
//              wave of each group of queries that holds the entry; every reader takes one off when it
//              is through): at zero the slot may be overwritten
//   next_load  entries are requested strictly in order, entry L into any slot that is free, by the waves
//              that are waiting for a tile: the one that notices first claims the slot with a compare-and-
//              swap and the entry with an add, waits for the load (it is idle anyway, or at the top of its next trip) and
//              publishes it.  Waves that have a tile to work on do not look for room.
// (With entry L tied to slot L % 8, one slow reader of entry L - 8 kept the others waiting whatever else was free: 24 heads x
// 1980 blocks 11.96 -> 11.77 ms, three heads of 65 frames 5.41 -> 5.31, 8 heads x 252 blocks stage by stage 319 -> 308 us; and
// requests four loads to a value of m0 instead of one, with a vector address each: 12.14 -> 11.96 ms, 5.50 -> 5.41, 324 -> 319.)
// A wave reads all of this with one LDS access per poll.  Every wait is bounded: if a tile does
// not show up the wave gives up (its output rows are then NaN, but the kernel always ends).
//
// V does not go through LDS.  After S = QK^T of a tile a wave knows the largest score of each of
// its queries; when every score of the tile is so far below the best the query has seen that
// all such keys of a row together weigh less than 2^-14 of its largest term, the tile cannot
// change the result at the precision of the output and its exponentials and second product are
// skipped.  With peaked attention that is the common case, so V^T operands are fetched from
// global memory (L2) straight into registers, only by the waves that need them, while the
// exponentials are being computed.
//
// The normaliser of a row is the sum of its probabilities as the second product sees them, i.e. after their
// rounding to bf16 (v_dot2c_f32_bf16 with a pair of ones: one instruction per two probabilities): numerator and
// denominator then carry the same rounding, and a row dominated by one key returns that key's V row exactly.
//
// The running max only moves (and O is rescaled) when a row max exceeds it by more than 2^8 in
// the exponent's units; until then probabilities are formed against the stale max, which is
// exact after the final division because numerator and denominator share it.  (Where a list is short, and in the first tiles of
// others, it follows the scores more closely: see the walk.)
#include <float.h>
#include <math.h>
#include <stdlib.h>
#include <string.h>
#include <type_traits>
#include "da_internal.h"
#include "ring_turns.h"

namespace da {
namespace ring {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) unsigned char* lds_bytes;
typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
typedef __attribute__((address_space(3))) int lds_int;

constexpr int D = 128;
constexpr int BS = 64;
constexpr int K_TILE = BS * D * 2;   // 16 KB, rows of 256 B
constexpr int V_TILE = D * BS * 2;   // 16 KB, rows of 128 B
constexpr int RING = 8;
constexpr int SLOT = K_TILE;
constexpr int RING_BYTES = RING * SLOT;           // 128 KB
constexpr int LDS_TOTAL = 160 * 1024;
static_assert(AUX_BYTES == LDS_TOTAL - RING_BYTES, "bitmaps + union list + ring state");
constexpr int WAVES = 8;
constexpr int O_STRIDE = D * 2 + 16;              // padded row stride of the output staging area
constexpr float kScale = 0.08838834764831845f;                      // 1/sqrt(128)
constexpr float kC2 = 0.08838834764831845f * 1.4426950408889634f;   // log2(e)/sqrt(128)
constexpr float kLazy = 8.0f;                     // move the running max only past this many powers of two
constexpr float kDropLog2 = 14.0f;                // all keys dropped from a row together weigh less than 2^-14 of its largest term
constexpr int kSpinLimit = 1 << 20;
constexpr int kClaimed = 1 << 20;                    // a slot's reader count while its entry is not known yet
constexpr int kMemberBit = 24;                       // fields of a union entry: the key sub-block below kValidBit, its valid keys, who wants it
constexpr int kPeekTiles = 8;                       // lists of at least so many tiles per wave: all waves of a group look at their own block first
constexpr int kFollowTiles = 24;                    // lists of fewer tiles, one wave each: the reference follows every larger score
constexpr int kNearTiles = 2;                       // and in so many tiles it is the largest of each 32 keys,
constexpr float kBelowTop = 90.0f;                  // no further below the largest score so far than this (11 powers of two)

// Waves whose bounded wait for a tile ran out since the library was loaded (their rows were written as NaN).
// No valid input makes that happen; the host can ask (da_wait_failures).
__device__ unsigned long long g_wait_failures = 0ull;

// ---------------------------------------------------------------------------------- tile movement
// 16 KB tile, rows of ROWB bytes, moved 1 KB (64 lanes x 16 B) per step; step `it` covers rows
// it*RPS .. it*RPS+RPS-1 (RPS*ROWB = 1024), so global and LDS offsets are both it*1024 plus a
// per-lane part that only depends on it & 3.
template <int ROWB>
__device__ inline void tile_lane_offsets(int lane, unsigned loff[4]) {
  constexpr int CPR = ROWB / 16;
  constexpr int RPS = 64 / CPR;
  const int r_in = lane / CPR, p = lane % CPR;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    int row = a * RPS + r_in;
    int sw = ROWB == 256 ? (row & 15) : ((row >> 1) & 7);
    loff[a] = r_in * ROWB + ((p ^ sw) << 4);
  }
}

// Direct-to-LDS load of 16 bytes per lane: lane i's data lands at m0 + 16*i.  m0 is put back afterwards (the
// load has read it by then), so whatever the compiler keeps in it across this statement survives.
__device__ __forceinline__ void dma16(const unsigned char* g, unsigned lds_addr) {
  unsigned keep;
  asm volatile(
      "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\ts_mov_b32 m0, %0"
      : "=&s"(keep)
      : "v"(g), "s"(lds_addr)
      : "memory");
}
// The same for a tile, four loads to a value of m0 (the instruction's offset counts on both sides).
__device__ __forceinline__ void dma_tile(const unsigned char* src, unsigned lds_addr, const unsigned (&loff)[4]) {
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    unsigned keep;
    asm volatile(
        "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %6\n\ts_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %5\n\t"
        "global_load_lds_dwordx4 %2, %5 offset:1024\n\t"
        "global_load_lds_dwordx4 %3, %5 offset:2048\n\t"
        "global_load_lds_dwordx4 %4, %5 offset:3072\n\ts_mov_b32 m0, %0"
        : "=&s"(keep)
        : "v"(loff[0]), "v"(loff[1]), "v"(loff[2]), "v"(loff[3]), "s"(src + b * 4096), "s"(lds_addr + b * 4096)
        : "memory");
  }
}
__device__ __forceinline__ void wait_vm0() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// the lane number, in a way that the compiler neither moves nor keeps
__device__ __forceinline__ int opaque_lane() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

// minus infinity, not kept in a register
__device__ __forceinline__ float opaque_minus_inf() {
  float x;
  asm volatile("v_mov_b32 %0, 0xff800000" : "=v"(x));
  return x;
}

__device__ inline int sigma(int r) { return (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1); }

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------------------------- softmax pieces
__device__ __forceinline__ float max16(const f32x16& a, float m) {
#pragma unroll
  for (int i = 0; i < 16; i += 2) m = fmaxf(fmaxf(a[i], a[i + 1]), m);   // v_max3_f32
  return m;
}

// max with the other half-wave's lane (l ^ 32): one v_permlane32_swap
__device__ __forceinline__ float max_across_halves(float x) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_across_halves(float x) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// exp / sum / pack of two scores (registers o, o + 1 of an accumulator tile) into elements e, e + 1 of a P operand
__device__ __forceinline__ void exp_pair(const f32x16& s, int o, float mc, float& lsum, bf16x8& p, int e) {
  const bf16x2 kOnes = {(__bf16)1.0f, (__bf16)1.0f};
  float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[o], kC2, -mc));
  float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[o + 1], kC2, -mc));
  f32x2 pp = {p0, p1};
  bf16x2 pb = __builtin_convertvector(pp, bf16x2);
  lsum = __builtin_amdgcn_fdot2_f32_bf16(pb, kOnes, lsum, false);   // the sum of what the second product sees
  p[e] = pb[0];
  p[e + 1] = pb[1];
}

// pad keys out of the softmax: accumulator register i is key 16(i>>3) + 8hh + (i&7) of the half tile, nv of its keys are valid
__device__ __forceinline__ void mask_pad_keys(f32x16& s, int nv) {
  const int lim = nv - ((opaque_lane() >> 5) << 3);
  const float ninf = opaque_minus_inf();
#pragma unroll
  for (int i = 0; i < 16; ++i) s[i] = 16 * (i >> 3) + (i & 7) < lim ? s[i] : ninf;
}

// n / d for 0 <= n < 2^27, d >= 1, n / d < 2^20, by way of the float reciprocal (exact: the estimate is off by one at most)
__device__ __forceinline__ int small_div(int n, int d) {
  int qt = (int)((float)n * __frcp_rn((float)d));
  const int rem = n - qt * d;
  qt += rem >= d ? 1 : 0;
  qt -= rem < 0 ? 1 : 0;
  return qt;
}

// how many lanes below this one are set in m
__device__ __forceinline__ int lanes_before(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0));
}

// valid slots of block j (blocks are numbered below 2^18)
__device__ __forceinline__ int valid_slots(const Geo& q, int per_frame, int j) {
  const int rr = j - small_div(j, per_frame) * per_frame;
  const int bi = small_div(rr, q.gw), bj = rr - bi * q.gw;
  return min(q.ph, q.fh - bi * q.ph) * min(q.pw, q.fw - bj * q.pw);
}

struct Soft {
  // Reference (raw score units): a maximum of some of the scores.  Before the first tile the lowest finite value and not minus infinity: all scores of a
  // half tile may be minus infinity (finite operands whose product leaves the range), and those keys weigh exp2(-inf) = 0,
  // not exp2(-inf + inf).
  float m;
  // Largest score seen so far, in what was carried out and in a tile that was only looked at; +inf for a pad query.  (The
  // reference trails the scores the wave has carried out by at most kLazy powers of two, or by kBelowTop in the first tiles of
  // a short list; it may start up to the drop rule's cut below a score that was only looked at.)
  float top;
  float l;     // this lane's partial sum of probabilities
};

__device__ __forceinline__ bf16x8 lds_operand(unsigned addr) { return *(const lds_bf16x8*)(uintptr_t)addr; }

// 16 bytes per lane from a uniform base
__device__ __forceinline__ bf16x8 load_operand(__amdgpu_buffer_rsrc_t base, unsigned lane_offset, unsigned offset) {
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(base, lane_offset, offset, 0);
  return __builtin_bit_cast(bf16x8, x);
}

// NQ: how many of the wave's two tiles of 32 queries are worked on (1 where the second holds nothing but pad slots)

// The scores of 32 keys against the wave's queries, S^T = K Q^T.  kaddr: this lane's LDS address of the operand of k-step
// 0; the swizzle puts that of step t at kaddr ^ 32t.
template <int NQ>
__device__ __forceinline__ void half_scores(unsigned kaddr, int nv, const bf16x8 (&qf)[2][8], f32x16 (&s)[NQ]) {
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  constexpr int AHEAD = 3;                            // operands on their way from LDS
  bf16x8 k[8];
#pragma unroll
  for (int t = 0; t < AHEAD; ++t) k[t] = lds_operand(kaddr ^ (32 * t));
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int t = 0; t < 8; ++t) {
#pragma unroll
    for (int h = 0; h < NQ; ++h) s[h] = mfma(k[t], qf[h][t], t == 0 ? zero : s[h]);
    if (t + AHEAD < 8) k[t + AHEAD] = lds_operand(kaddr ^ (32 * (t + AHEAD)));
    __builtin_amdgcn_sched_barrier(0);
  }
  if (nv < 32) {
#pragma unroll
    for (int h = 0; h < NQ; ++h) mask_pad_keys(s[h], nv);
  }
}

// 32 keys (half a tile) for one wave.  lazy: how many powers of two the reference may trail the scores by; minus infinity: it
// becomes the largest of these 32, also where that is smaller.  v: the half tile's V^T in global memory (operand order: the 64 lanes' operands of
// (k-step t, channel group dt) are the contiguous KB number 4t + dt, so every load of a wave is one contiguous KB).
template <int NQ>
__device__ __forceinline__ void half_tile(unsigned kaddr, const unsigned char* v, int nv, float skip, float lazy,
                                          const bf16x8 (&qf)[2][8], f32x16 (&o)[2][4], Soft (&st)[2], int& kept) {
  f32x16 s[NQ];
  half_scores<NQ>(kaddr, nv, qf, s);
  // online softmax over the 32 keys
  float mx[NQ];
  bool negligible = true;
#pragma unroll
  for (int h = 0; h < NQ; ++h) {
    mx[h] = max_across_halves(max16(s[h], -INFINITY));
    negligible = negligible && (mx[h] - st[h].top) * kC2 < -skip;
  }
  // A key whose score is more than `skip` powers of two below the query's best score so far
  // weighs less than 2^-skip of that query's largest term, in the normaliser and in the output.
  // skip = log2(keys in the row) + kDropLog2, so whatever is dropped from a row adds up to less
  // than 2^-kDropLog2 of that term: below the resolution of a bf16 result at any sequence length.
  // When all 32 keys are that small for every query, the exponentials and the second
  // product are skipped.  (Never while top is -inf, unless all 32 scores are.)  Pad query slots have no say (their top is
  // +inf): their rows are zero, every score is 0, and nobody reads their output.
  if (__all(negligible)) return;
  __builtin_amdgcn_s_setprio(1);
  asm volatile("s_add_u32 %0, %0, 1" : "+s"(kept) : : "scc");   // (a scalar, whatever the compiler thinks)
  // V^T operands: the first three on their way while the exponentials are computed, one more whenever registers fall
  // free.  (Operand 4t + dt belongs to k-step t and channel group dt.)
  const __amdgpu_buffer_rsrc_t vb = __builtin_amdgcn_make_buffer_rsrc((void*)v, 0, -1, 0x00020000);
  const unsigned lane16 = (unsigned)(opaque_lane() & 63) * 16;
  bf16x8 va[8];
  auto fetch = [&](int i) { va[i] = load_operand(vb, lane16 + (i & 3) * 1024, (i >> 2) * 4096); };
  fetch(0);
  fetch(1);
  fetch(2);
  __builtin_amdgcn_sched_barrier(0);
  bool moves = false;
#pragma unroll
  for (int h = 0; h < NQ; ++h) {
    st[h].top = fmaxf(st[h].top, mx[h]);
    moves = moves || (mx[h] - st[h].m) * kC2 > lazy;
  }
  if (__any(moves)) {
#pragma unroll
    for (int h = 0; h < NQ; ++h) {
      const bool near = lazy < 0.f && st[h].top < INFINITY;              // (not for pad queries)
      const float m_new = fmaxf(near ? fmaxf(st[h].top - kBelowTop, -FLT_MAX) : st[h].m, mx[h]);
      const float alpha = st[h].m == m_new ? 1.0f : __builtin_amdgcn_exp2f((st[h].m - m_new) * kC2);   // 0 the first time
      st[h].m = m_new;
      st[h].l *= alpha;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[h][dt][i] *= alpha;
    }
  }
  bf16x8 p[NQ];
#pragma unroll
  for (int h = 0; h < NQ; ++h) {
#pragma unroll
    for (int i = 0; i < 8; i += 2) exp_pair(s[h], i, st[h].m * kC2, st[h].l, p[h], i);
    __builtin_amdgcn_sched_barrier(0);
    fetch(3 + h);
    __builtin_amdgcn_sched_barrier(0);
  }
  // O^T += V^T P^T.  The second half of the probabilities is made between the first half's matrix instructions, a pair
  // after each: the wave has vector work while the pipe is busy and need not find a partner that has.  Together with the
  // raised priority (from here to the end of the tile a wave is in the way of nobody who waits for V or a tile; neither is
  // worth 1 % alone), nothing dropped: 8x16 windows 20.2 -> 19.6 ms, 5 heads x 1260 blocks 4.79 -> 4.66 ms, dense 480p 2.00 ->
  // 1.94 ms.  24 heads x 1980 blocks (21.1 -> 20.9 ms) and peaked inputs change by no more than two runs of one side differ.
  bf16x8 p2[NQ];
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) {
#pragma unroll
    for (int h = 0; h < NQ; ++h) {
      o[h][dt] = mfma(va[dt], p[h], o[h][dt]);
      __builtin_amdgcn_sched_barrier(0);
      exp_pair(s[h], 8 + 2 * dt, st[h].m * kC2, st[h].l, p2[h], 2 * dt);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (3 + NQ + dt < 8) fetch(3 + NQ + dt);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int h = 0; h < NQ; ++h) o[h][dt] = mfma(va[4 + dt], p2[h], o[h][dt]);
  __builtin_amdgcn_s_setprio(0);
}

// Puts the n union entries at `list` in the order of the walk (see there), by all eight waves.  The scratch is the ring's place,
// which holds nothing yet; ends with a barrier.  Number within the class: a wave takes a stretch of the list, 64 entries at a
// time; rank by key: kWalkBuckets buckets of keys, and inside a bucket by comparison (whatever the order in which waves reach
// the counters, the result is the same).  An entry's key is formed once and read back from then on: the passes have to agree on
// its bucket, for one more entry in a bucket than were counted would take the place of another.
__device__ __forceinline__ void spread_walk(unsigned char* scratch, unsigned* list, int n, int wave, int lane) {
  int* const of_class = (int*)scratch;                // [WAVES][256] entries of a class in each wave's stretch, then before it
  float* const inv_total = (float*)(scratch + 8192);  // [256]
  int* const next = (int*)(scratch + 16384);          // [kWalkBuckets] entries per bucket, then where its next one goes: in the end where the next bucket starts
  int* const wave_sum = (int*)(scratch + 28672);      // [WAVES]
  int* const number = (int*)(scratch + 32768);        // [n] number within the stretch's part of the class, then the key
  uint2* const slots = (uint2*)(scratch + 65536);     // [n] key and entry
  const int t = threadIdx.x;
  for (int i = t; i < WAVES * 256; i += 512) of_class[i] = 0;
  for (int i = t; i < kWalkBuckets; i += 512) next[i] = 0;
  __syncthreads();
  const int stretch = ((n + 511) >> 9) << 6;
  for (int base = wave * stretch; base < min(n, (wave + 1) * stretch); base += 64) {
    const int i = base + lane;
    const int m = i < n ? (int)(list[i] >> kMemberBit) : 0;
    unsigned long long same = ~0ull;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const unsigned long long has = __ballot((m >> b) & 1);
      same &= (m >> b) & 1 ? has : ~has;
    }
    const int before = lanes_before(same), c = of_class[wave * 256 + m];
    if (i < n) number[i] = c + before;
    asm volatile("" ::: "memory");
    if (before == 0) of_class[wave * 256 + m] = c + __popcll(same);
    asm volatile("" ::: "memory");
  }
  __syncthreads();
  if (t < 256) {
    int sum = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const int c = of_class[w * 256 + t];
      of_class[w * 256 + t] = sum;
      sum += c;
    }
    inv_total[t] = 1.0f / (float)max(sum, 1);
  }
  __syncthreads();
  for (int i = t; i < n; i += 512) {
    const int m = (int)(list[i] >> kMemberBit);
    const float key = walk_key(m, number[i] + of_class[(i / stretch) * 256 + m], inv_total[m]);
    number[i] = __float_as_int(key);
    atomicAdd(&next[walk_bucket(key)], 1);
  }
  __syncthreads();
  {
    int c[4], sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      c[j] = sum;
      sum += next[4 * t + j];
    }
    int incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int x = __shfl_up(incl, o);
      incl += lane >= o ? x : 0;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int at = incl - sum;
    for (int w = 0; w < wave; ++w) at += wave_sum[w];
#pragma unroll
    for (int j = 0; j < 4; ++j) next[4 * t + j] = at + c[j];
  }
  __syncthreads();
  for (int i = t; i < n; i += 512) {
    const int key = number[i];
    slots[atomicAdd(&next[walk_bucket(__int_as_float(key))], 1)] = make_uint2((unsigned)key, list[i]);
  }
  __syncthreads();
  for (int i = t; i < n; i += 512) {
    const uint2 mine = slots[i];
    const float key = __uint_as_float(mine.x);
    const int bucket = walk_bucket(key), lo = bucket ? next[bucket - 1] : 0, hi = next[bucket];
    int rank = lo;
    for (int x = lo; x < hi; ++x) {
      const uint2 other = slots[x];
      const float its = __uint_as_float(other.x);
      rank += its < key || (its == key && other.y < mine.y) ? 1 : 0;
    }
    list[rank] = mine.y;
  }
  __syncthreads();
}

// SUB = 64-token sub-blocks per block (1: 8x8 patches, 2: 128-token blocks such as 8x16 patches).  A block of
// 128 is two K tiles and two V tiles in a row, and its queries are two waves' worth: the workgroup then takes four
// query blocks (four consecutive frames) instead of eight, and a key block enters the union walk as two entries.
// LISTS: the kept blocks come as lists of any length (row_ptr) instead of k per row.
template <int SUB, bool LISTS>
__global__ __launch_bounds__(512, 2) void attn_bf16_ring_kernel(Geo q, const unsigned char* __restrict__ Qp,
                                                               const unsigned char* __restrict__ Kp,
                                                               const unsigned char* __restrict__ Vt,
                                                               const int32_t* __restrict__ idx,
                                                               const int32_t* __restrict__ row_ptr, long long cap,
                                                               unsigned char* __restrict__ Op, float* __restrict__ lse,
                                                               float skip, int direct, Share share,
                                                               unsigned long long* __restrict__ tile_counts) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[LDS_TOTAL];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int lane = threadIdx.x & 63;
  // Heads one after the other (the K/V of the heads in flight then fit the last-level cache); inside a head a unit is one
  // patch position and FG consecutive frames (or left-over frames of a few positions: unit_place).  Units are dealt to the 8 XCDs in
  // turn, as workgroups are; only the shares of one unit stay together on one.
  constexpr int LOG_FG = SUB == 1 ? 3 : 2;
  constexpr int FG = 1 << LOG_FG;                     // query blocks (frames) per unit
  constexpr int BLOCK = BS * SUB;                     // slots per block
  const int per_frame = q.gh * q.gw;
  const int per_head = units_per_head(q.T, FG, per_frame);
  // The eight groups of 64 queries of a unit are shared between 2^lsub workgroups, with 2^lsub waves to a group.
  const ShareOf mine_is = share_of(share, (int)blockIdx.x, per_head, left_units(q.T, FG, per_frame));
  const int lsub = mine_is.lsub, sub = mine_is.sub;
  const long long bh = mine_is.head;
  if (bh >= (long long)q.B * q.H) return;             // (the last eight units need not be eight)
  const UnitPlace place = unit_place(mine_is.unit, q.T, LOG_FG, per_frame);
  // waves w and w+4 share a SIMD: they have different groups where there are some.
  // The waves of a group take its list entries in turn (part = which of them).
  const int groups = 8 >> lsub, parts = 1 << lsub;
  const int part = wave >> (3 - lsub);
  const int lgroup = (wave + (wave >> 2) * (lsub ? 3 - lsub : 0)) & (groups - 1);   // number of the group in this workgroup
  const int group = sub * groups + lgroup;            // and in the unit
  const int qsub = SUB == 1 ? 0 : group & 1;          // which 64 queries of the block
  const int first_slot = sub * groups / SUB;          // query blocks of this workgroup: so many from this one on
  const int blocks = max(groups / SUB, 1);
  const int lblock = group / SUB - first_slot;        // my query block's number among them
  // block number of query block w of this workgroup, -1 if the place is empty (then all after it are)
  auto slot_block = [&](int w) -> int {
    const int p = unit_pos(place, first_slot + w), fr = unit_frame(place, first_slot + w);
    return w < blocks && p < per_frame ? fr * per_frame + p : -1;
  };
  if (slot_block(0) < 0) return;                      // past the last position
  const int my_block = slot_block(lblock);
  const bool has_block = my_block >= 0;
  // a wave without a query block, or whose 64 slots of it are all pad slots, takes no tiles
  const int q_valid = (has_block ? block_valid(q, my_block) : 0) - BS * qsub;   // valid queries of the group
  const bool live = q_valid > 0;
  const long long qb = bh * q.g + (has_block ? my_block : 0);
  const int g = q.g;
  // The list of my query block: k columns at idx + (row) * k, or, with row_ptr (lists of any length, one head's
  // after the other in a stretch of `cap` entries), the columns between two offsets.
  int k = q.k;
  const int32_t* list = idx + qb * k;
  if (LISTS) {
    const int32_t* rp = row_ptr + bh * (g + 1) + (has_block ? my_block : 0);
    // (offsets that are not what the interface asks for are brought into the head's stretch: such lists give
    // unspecified results, but nothing outside the arrays is read)
    const int begin = min(max(rp[0], 0), (int)cap);
    list = idx + bh * cap + begin;
    k = min(max(rp[1] - begin, 0), (int)cap - begin);
    // the cut of the drop rule goes by the number of keys in this row
    skip = log2f((float)max(k, 1) * (float)BLOCK) + kDropLog2;
  }

  // The first 256 entries of the lists are asked for before anything else: everything up to the walk waits for them.
  const bool lister = live && part == 0 && (qsub == 0 || groups == 1); // the wave that brings in the list of its query block
  int pre[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) pre[i] = lister && lane + 64 * i < k ? list[lane + 64 * i] : -1;
  __builtin_amdgcn_sched_barrier(0);

  // With `direct`, Qp and Op are the caller's Q and O (q.in, q.out: in the original token order as a rule): the
  // reordering of Q and the restoring of O (Algorithms 1 and 2) are then this kernel's addressing, slot -> row.
  const BlockPos qpos = block_pos(q, has_block ? my_block : 0);
  const long long q_first = block_first_row(q, has_block ? my_block : 0, qpos);
  const int q_pitch = block_row_pitch(q, qpos);
  // slots of my query block with a row of their own there (a pad slot has none in the original order)
  const int rows_there = direct ? qpos.vh * qpos.vw : BLOCK;
  // where the row of slot 0 of my query block is, in bytes, and how many bytes slot s lies behind it
  auto row_base = [&](const Rows& where) -> long long {
    return 2 * (direct ? row_offset(where, q.H, bh, q_first) : qb * BLOCK * (long long)D);
  };
  auto row_after = [&](const Rows& where, int s, bool there) -> long long {
    if (!there) return s * (D * 2);
    const int u = (s * ((65536 + qpos.vw - 1) / qpos.vw)) >> 16;   // s / vw by way of the reciprocal: exact below 256
    return (long long)(u * (q_pitch - qpos.vw) + s) * (where.sn * 2);
  };

  unsigned* bitmap = (unsigned*)(smem + RING_BYTES);  // [blocks][bw] one bitmap of kept key blocks per query block
  const int bw = (g + 31) >> 5;
  unsigned* ulist = bitmap + blocks * bw;             // union entries: key sub-block | (valid slots - 1) << 18 | membership << 24
  int* ctrl = (int*)(smem + LDS_TOTAL - 128);         // [32]: ready[8], left[8], next_load, count[2], mixed, (1 unused), wcount[8], live groups, waves that gave up
  int* ready = ctrl;                                  // [RING]
  int* left = ctrl + 8;                               // [RING]
  int* next_load = ctrl + 16;
  int* count = ctrl + 17;                             // [2]

  // ---- union of the workgroup's lists
  for (int i = threadIdx.x; i < blocks * bw; i += 512) bitmap[i] = 0u;
  if (threadIdx.x < 32) ctrl[threadIdx.x] = threadIdx.x < RING ? -1 : 0;
  __syncthreads();
  if (live && part == 0 && lane == 0) atomicOr(&ctrl[28], 1 << lgroup);   // which groups take tiles at all
  if (lister) {
    // (an entry that is no block number is left out: it must not reach the bitmap, let alone an address)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if ((unsigned)pre[i] < (unsigned)g) atomicOr(&bitmap[lblock * bw + (pre[i] >> 5)], 1u << (pre[i] & 31));
    for (int e = lane + 256; e < k; e += 64) {
      int j = list[e];
      if ((unsigned)j < (unsigned)g) atomicOr(&bitmap[lblock * bw + (j >> 5)], 1u << (j & 31));
    }
  }
  // Q comes in by way of the ring, which is empty until the walk: 64 rows per group in a slot, as a K tile lies there, the
  // rows dealt to the group's waves.  (Every wave for itself and straight to registers, 64 rows are twice the bytes and 16 loads
  // that touch 32 rows each: asking for them took 1.4 to 1.9 us of a workgroup, 0.5 with 32 queries per wave.  da_forward, 48
  // heads, one 48x80 frame with 5 % kept 146 -> 138 us, four frames 691 -> 663 us; one 30x52 frame, half kept, 122.4 -> 119.8 us.)
  const unsigned ring_lds = (unsigned)(uintptr_t)(lds_bytes)smem;
  const unsigned q_lds = ring_lds + (unsigned)lgroup * SLOT;
  if (live) {
    const unsigned char* const q0 = Qp + row_base(q.in);
    for (int it = part; it < 16; it += parts) {
      const int row = 4 * it + (lane >> 4);
      const int slot = min(BS * qsub + row, rows_there - 1);   // (what has no row of its own is zeroed below)
      dma16(q0 + row_after(q.in, slot, direct) + (((lane & 15) ^ (row & 15)) << 4), q_lds + it * 1024);
    }
  }
  __syncthreads();
  // The workgroup's own blocks go first (when kept): a query's best scores tend to be
  // there, and the sooner the running maximum is near its final value, the more of the other
  // tiles turn out negligible.
  int own_j[FG];                                      // the workgroup's own blocks (-1: empty slot)
#pragma unroll
  for (int w = 0; w < FG; ++w) own_j[w] = slot_block(w);
  // membership of key block j in the workgroup's lists (0 for the own blocks unless asked for)
  auto membership = [&](int j, bool want_own) -> unsigned {
    bool own = false;
#pragma unroll
    for (int w = 0; w < FG; ++w) own = own || j == own_j[w];
    unsigned m = 0;
    if (j < g && own == want_own)
      for (int w = 0; w < blocks; ++w) m |= ((bitmap[w * bw + (j >> 5)] >> (j & 31)) & 1u) << w;
    return m;
  };
  // a key block becomes one entry per 64-slot sub-block that holds a valid slot (in a row)
  auto second = [&](int j) -> bool { return SUB == 2 && j < g && valid_slots(q, per_frame, j) > BS; };
  auto put_entries = [&](int at, int j, unsigned m, bool two) {
    const int nvb = valid_slots(q, per_frame, j);
    ulist[at] = (unsigned)(j * SUB) | ((unsigned)(min(nvb, BS) - 1) << kValidBit) | (m << kMemberBit);
    if (two) ulist[at + 1] = (unsigned)(j * SUB + 1) | ((unsigned)(nvb - BS - 1) << kValidBit) | (m << kMemberBit);
  };
  // every wave takes a contiguous eighth of the key blocks, 64 at a time: count, then place
  int* wcount = ctrl + 20;                            // [WAVES]
  const int chunks = (g + 63) >> 6, cpw = (chunks + WAVES - 1) / WAVES;
  const int c_lo = wave * cpw, c_hi = min(chunks, c_lo + cpw);
  {
    int cnt = 0;
    if (SUB == 1) {
      // one entry per key block in any list: count the bits of the OR of the bitmaps, word by word
      // (lane l takes word l of the wave's range), minus the own blocks among them
      const int w_lo = 2 * c_lo, w_hi = min(2 * c_hi, bw);
      for (int base = w_lo; base < w_hi; base += 64) {
        const int word = base + lane;
        unsigned v = 0u;
        if (word < w_hi) {
          for (int w = 0; w < blocks; ++w) v |= bitmap[w * bw + word];
#pragma unroll
          for (int w = 0; w < FG; ++w)
            if (own_j[w] >= 0 && (own_j[w] >> 5) == word) v &= ~(1u << (own_j[w] & 31));
        }
        int pop = __popc(v);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) pop += __shfl_xor(pop, o);
        cnt += pop;
      }
    } else {
      for (int c = c_lo; c < c_hi; ++c) {
        const int j = c * 64 + lane;
        const bool in = membership(j, false) != 0u;
        cnt += __popcll(__ballot(in)) + __popcll(__ballot(in && second(j)));
      }
    }
    if (lane == 0) wcount[wave] = cnt;
    if (wave == 0) {
      int j = -1;
#pragma unroll
      for (int w = 0; w < FG; ++w) j = lane == w ? own_j[w] : j;
      const unsigned m = j >= 0 ? membership(j, true) : 0u;
      const bool two = m != 0u && second(j);
      const unsigned long long nz = __ballot(m != 0u), n2 = __ballot(two);
      if (m) put_entries(lanes_before(nz) + lanes_before(n2), j, m, two);
      if (lane == 0) count[1] = __popcll(nz) + __popcll(n2);
    }
  }
  wait_vm0();                                         // (my share of Q has landed)
  __syncthreads();
  // Q fragments (B operand): lane (query r, half-wave hh) holds d = 16t + 8hh .. +7.  (Read by all before the first tile is
  // asked for: barriers lie between.)
  bf16x8 qf[2][8];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int row = 32 * h + (lane & 31);
    const unsigned at = q_lds + row * 256 + (((lane >> 5) ^ (row & 15)) << 4);
#pragma unroll
    for (int t = 0; t < 8; ++t) qf[h][t] = lds_operand(at ^ (32 * t));
    if (direct && row >= q_valid) {
#pragma unroll
      for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int i = 0; i < 8; ++i) qf[h][t][i] = (__bf16)0.f;
    }
  }
  {
    int at = count[1];
    for (int w = 0; w < wave; ++w) at += wcount[w];
    unsigned all = 0;
    for (int w = 0; w < blocks; ++w) all |= slot_block(w) >= 0 ? 1u << w : 0u;
    bool some = false;
    for (int c = c_lo; c < c_hi; ++c) {
      const int j = c * 64 + lane;
      const unsigned m = membership(j, false);
      const bool two = m != 0u && second(j);
      const unsigned long long nz = __ballot(m != 0u), n2 = __ballot(two);
      if (m) put_entries(at + lanes_before(nz) + lanes_before(n2), j, m, two);
      at += __popcll(nz) + __popcll(n2);
      some = some || (m != 0u && m != all);
    }
    if (some) ctrl[19] = 1;
    if (wave == WAVES - 1 && lane == 0) count[0] = at;
  }
  __syncthreads();
  const int nU = __builtin_amdgcn_readfirstlane(count[0]);
  const int n_own = __builtin_amdgcn_readfirstlane(count[1]);
  const bool mixed = __builtin_amdgcn_readfirstlane(ctrl[19]) != 0;   // not every block of the workgroup keeps every entry

  // ---- order of the walk.  In ascending order the blocks' shares of the work come in runs (the earliest frames of the
  // union only matter to the first block, the latest only to the last), and since nobody can run more than RING entries
  // ahead, waves would take turns waiting.  Entries with the same membership form a class, and each class is spread evenly
  // over the walk: number p of the c entries of class m gets the key (p + u)/c, u the fraction of m times the golden
  // section (so that the classes of one or two entries spread as well), and the walk goes by ascending key.  Every stretch
  // of it then holds every block's fair share.  The softmax does not care about the order of the keys.
  if (mixed && nU - n_own > 2 * RING) spread_walk(smem, ulist + n_own, nU - n_own, wave, lane);

  // A group's own block is the best start for its running maxima.  One of the group's waves takes it in its turn; the others look
  // at its scores before they start, so that none has to carry out tiles that the drop rule would spare it.  Not worth a product
  // where a wave has few tiles.  A list without it: the group's first entry.  (The own blocks are the first entries of the walk, eight
  // at most, so all of them are in the ring before anybody has to be through with one.  Looking at the group's first entry in any
  // case leaves all but one wave without a good start where the unit's blocks are of several positions, as those of left-over
  // frames are: dense, peaked, one head x 760 blocks of 19 frames 888 -> 592 us, 3 heads x 196 of 7 253 -> 190 us, 8 x 84 of 3 121 ->
  // 102 us; 405 of 15 frames, half kept, 301 -> 250 us.  Where attention is not peaked it makes no difference.)
  const bool few = k * SUB < kPeekTiles * parts;
  const unsigned my_bit = live ? (1u << (kMemberBit + lblock)) : 0u;
  const unsigned my_entry = (unsigned)(my_block * SUB + qsub);        // (not met where the group has no block)
  constexpr int kTaker = 20;                          // the field of `first` that says which wave takes it
  int* first = wcount;                                // [groups] that entry of each group and who takes it, -1: nobody looks
  {
    int f = -1;
    if (live && !few && parts > 1)
      for (int base = 0; base < nU; base += 64) {
        const unsigned e = ulist[min(base + lane, nU - 1)];
        const unsigned long long ours = __ballot(base + lane < nU && (e & my_bit) != 0u);
        if (ours) {
          const unsigned long long own = __ballot((e & ((1u << kValidBit) - 1u)) == my_entry) & (base ? 0ull : ours);
          const int i = (int)__builtin_ctzll(own ? own : ours);
          f = (base + i) | wave_of_turn(__popcll(ours & ((1ull << i) - 1ull)), SUB, parts) << kTaker;
          break;
        }
      }
    if (part == 0 && lane == 0) first[lgroup] = f;
  }
  __syncthreads();

  // ---- per-lane constants
  const int krow = sigma(lane & 31);
  const unsigned kbase = ring_lds + krow * 256 + (((lane >> 5) ^ (krow & 15)) << 4);   // K operand of k-step 0 in slot 0, swizzle applied
  const unsigned char* Kbh = Kp + bh * q.n_pad * (D * 2);
  const unsigned char* Vbh = Vt + bh * q.n_pad * (D * 2);
  const int live_groups = __builtin_amdgcn_readfirstlane(ctrl[28]);
  int first_of[4];                                    // (where a group has one wave nobody looks)
#pragma unroll
  for (int w = 0; w < 4; ++w) first_of[w] = __builtin_amdgcn_readfirstlane(first[w]) & ((1 << kTaker) - 1);
  // one wave brings the K tile of union entry u into the given slot of the ring
  auto issue_tile = [&](int u, int slot) {
    const unsigned e = (unsigned)__builtin_amdgcn_readfirstlane((int)ulist[u]);
    // how many waves will read the tile: one of each live group that holds the entry, and the others where they look
    const int m = (int)(e >> kMemberBit);
    const int holds = live_groups & (SUB == 1 ? m : 3 * ((m & 1) | (m & 2) << 1 | (m & 4) << 2 | (m & 8) << 3));
    int readers = __builtin_popcount(holds);
#pragma unroll
    for (int w = 0; w < 4; ++w) readers += u == first_of[w] ? ((holds >> w) & 1) * (parts - 1) : 0;
    if (lane == 0) __atomic_store_n(&left[slot], readers, __ATOMIC_RELAXED);   // (before the transfer, hence before the slot is published)
    const long long j = (long long)(e & ((1u << kValidBit) - 1u));
    unsigned koff[4];
    tile_lane_offsets<256>(opaque_lane(), koff);      // (made anew each time: four registers the tile loop can use)
    dma_tile(Kbh + j * K_TILE, ring_lds + (unsigned)slot * SLOT, koff);
  };
  int pending = -1;                                   // entry I have asked for, and the slot it goes to
  int pending_slot = 0;
  // a tile this wave has requested becomes visible to the others once it has landed
  auto publish = [&]() {
    const int pd = __builtin_amdgcn_readfirstlane(pending);   // (the same in every lane; says so to the compiler)
    if (pd >= 0) {
      wait_vm0();
      if (lane == 0) __atomic_store_n(&ready[__builtin_amdgcn_readfirstlane(pending_slot)], pd, __ATOMIC_RELAXED);
      pending = -1;
    }
  };

  f32x16 o[2][4];
  Soft st[2];
  float nought;                                       // (a zero of its own: the compiler would keep a row of them for later uses)
  asm volatile("v_mov_b32 %0, 0" : "=v"(nought));
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[h][dt][i] = nought;
    st[h].m = -FLT_MAX;
    st[h].top = 32 * h + (lane & 31) < q_valid ? -INFINITY : INFINITY;
    st[h].l = nought;
  }
  // The Q fragments are in by here, and the compiler is to know: else it would wait for them at their first use inside the
  // tile loop, on every trip.
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int t = 0; t < 8; ++t) asm volatile("" : "+v"(qf[h][t]));

  // a look at the whole control block: lane i holds ctrl[i]
  const unsigned ctrl_lds = ring_lds + LDS_TOTAL - 128;
  auto look = [&]() -> int {
    unsigned at = (unsigned)(opaque_lane() & 31) * 4;
    asm volatile("v_add_u32 %0, %1, %0" : "+v"(at) : "s"(ctrl_lds));   // (as one constant it would be kept in a register)
    return __atomic_load_n((const lds_int*)(uintptr_t)at, __ATOMIC_RELAXED);
  };
  // request the next tile if there is a free slot, judging by a look c (which may be old: then the
  // compare-and-swap fails or the room is underestimated, both harmless)
  auto service = [&](int c) {
    if (__builtin_amdgcn_readfirstlane(pending) >= 0) return;   // at most one request of mine in flight
    if (__builtin_amdgcn_readlane(c, 16) >= nU) return;
    const unsigned free = (unsigned)(__ballot(c == 0) >> 8) & ((1u << RING) - 1u);   // slots that nobody has yet to read
    if (!free) return;
    const int slot = __builtin_ctz(free);
    int got = 0;
    if (lane == 0) {
      got = atomicCAS(&left[slot], 0, kClaimed) == 0 ? atomicAdd(next_load, 1) : -1;
      if (got >= nU) __atomic_store_n(&left[slot], 0, __ATOMIC_RELAXED);
    }
    got = __builtin_amdgcn_readfirstlane(got);
    if (got < 0 || got >= nU) return;
    issue_tile(got, slot);
    pending = got;
    pending_slot = slot;
  };
  bool gave_up = false;
  int snap = look();
  // which slot of a look holds entry u (bit mask)
  auto slot_of = [&](int u) -> unsigned { return (unsigned)__ballot(snap == u) & ((1u << RING) - 1u); };
  // wait until entry u is in a slot, and say in which (-1: the bounded wait ran out)
  auto arrived = [&](int u) -> int {
    publish();                                        // my last request has had a whole tile's time to land
    unsigned in = slot_of(u);
    if (in) return __builtin_ctz(in);
    int spins = 0;
    for (;;) {
      snap = look();
      service(snap);
      in = slot_of(u);
      if (in) return __builtin_ctz(in);
      if (__builtin_amdgcn_readfirstlane(pending) >= 0) {
        publish();                                    // idle anyway: wait for my own request and hand it over
      } else {
        __builtin_amdgcn_s_sleep(1);
        if (++spins > kSpinLimit) return -1;
      }
    }
  };
  // my reads of a slot are complete: one reader less
  auto leave = [&](int slot) {
    wait_lds();
    if (lane == 0) atomicSub(&left[slot], 1);
  };
  const bool two = q_valid > 32;                      // else the second 32 queries are all pad slots
  // Tiles of 32 queries and 64 keys gone through and, from bit 16 on, half tiles carried out, the only half of a tile with at
  // most 32 valid keys for two (one scalar register, reported when the caller asks for the counts: the union has at most
  // AUX_BYTES / 4 = 2^13 entries, and a wave counts 2 and 4 for each)
  unsigned tally = 0u;
  int before = 0;                                     // entries of my group in the chunks before
  // How closely the reference follows the scores.  The probability of the key it is taken from is 1, which bf16 holds
  // exactly, and those just below it round better than those just above, so every reference that a row's sums are made up of saves
  // part of the error.  Two waves to a list have two, each with its own tiles; one wave to a list makes up for that:
  //   - it follows every larger score while the unit's own blocks go by, where a row's largest terms mostly are;
  //   - in lists of fewer than kFollowTiles it follows throughout, and in the first kNearTiles each 32 keys have their own.
  // With several waves to a list the first tile of short ones is followed.
  // Error against float64 over that of two waves to every list with short ones (of up to 15 tiles) followed in the first tile
  // (q scaled by 1, 1/4, 1/32; before this rule -> now): 48 heads of a 30x52 frame, 3 kept 1.005 -> 0.995, 1.018 -> 0.993, 1.026 -> 0.992, 14 kept
  // 1.010 -> 0.998, 1.027 -> 0.992, 1.013 -> 0.994, 21 kept 1.009 -> 0.996, 1.014 -> 0.979, 1.005 -> 0.994; nine such frames,
  // 63 kept 1.048 -> 0.990, 1.013 -> 0.977, 1.001 -> 0.996; 8x16 windows, 24 kept 1.049 -> 0.981, 1.018 -> 0.970, 1.002 -> 0.994.
  // Tried besides: short lists that only follow, up to 1.008; with one tile where each 32 keys have their own 1.003, with four
  // 1 to 2 % slower still.  Long ones that follow in the wave's own block alone, or have each 32 keys' own there, up to 1.013 and
  // 1.001, and no faster.  What it costs (da_forward, us): 14 kept 100.6 -> 102.6, 3 kept 65.4 -> 67.2; 24 heads x 1980 blocks, 198 kept, peaked
  // 11629 -> 11715, flat 19557 -> 19613.  (Worked out for each tile from what the rule goes by, which is then kept through the loop, 11835
  // and 19694, and 23 heads x 14 frames of 20x71, 8x16, half kept, 1734 against 1711.)
  auto walk = [&](auto queries) {
    constexpr int NQ = decltype(queries)::value;
    // (one number and a count of tiles: what the rule goes by need not be kept through the loop)
    const bool follow = parts == 1 && k * SUB < kFollowTiles;
    int lazy = __float_as_int(parts > 1 ? (few ? 0.f : kLazy) : follow ? -INFINITY : 0.f), until = parts > 1 ? 1 : kNearTiles;
    const int look_at = parts > 1 ? __builtin_amdgcn_readfirstlane(first[lgroup]) : -1;
    if (live && look_at >= 0 && part != look_at >> kTaker) {
      const int u = look_at & ((1 << kTaker) - 1);
      const int slot = arrived(u);
      gave_up = slot < 0;
      if (!gave_up) {
        const int nv = (int)((__builtin_amdgcn_readfirstlane((int)ulist[u]) >> kValidBit) & 63) + 1;
#pragma unroll 1
        for (int half = 0; half < 2 && 32 * half < nv; ++half) {
          f32x16 s[NQ];
          half_scores<NQ>(kbase + (unsigned)slot * SLOT + half * (SLOT / 2), nv - 32 * half, qf, s);
#pragma unroll
          for (int h = 0; h < NQ; ++h) st[h].top = fmaxf(st[h].top, max_across_halves(max16(s[h], -INFINITY)));
        }
        leave(slot);
      }
    }
    // The walk, 64 entries at a time: lane i holds entry base + i, a ballot tells which of them are my group's, a second
    // one which of those are mine (wave_of_turn: every other one, or fourth, or eighth).  Entries that are not mine cost nothing.
    for (int base = 0; base < nU && !gave_up; base += 64) {
      const int at = base + opaque_lane();
      const unsigned e_lane = ulist[min(at, nU - 1)];
      const bool is_ours = at < nU && (e_lane & my_bit) != 0u;
      const unsigned long long ours = __ballot(is_ours);
      unsigned long long mine = __ballot(is_ours && wave_of_turn(before + lanes_before(ours), SUB, parts) == part);
      before += __popcll(ours);
      if (parts == 1 && !follow && base == 0) {       // (the own blocks, eight at most, are the first entries)
        until = __popcll(mine & ((1ull << n_own) - 1ull));
        if (until == 0) lazy = __float_as_int(kLazy);
      }
      while (mine) {
        const int i = (int)__builtin_ctzll(mine);
        mine &= mine - 1;
        const int u = base + i;
        const int slot = arrived(u);
        if (slot < 0) {
          gave_up = true;
          break;
        }
        snap = look();                                // asked for now, used after the tile: its latency hides behind the tile
        const unsigned e = (unsigned)__builtin_amdgcn_readlane((int)e_lane, i);
        const int nv = (int)((e >> kValidBit) & 63u) + 1;
        const unsigned kaddr = kbase + (unsigned)slot * SLOT;
        const unsigned char* v = Vbh + (long long)(e & ((1u << kValidBit) - 1u)) * V_TILE;
        int kept = 0;
#pragma unroll 1
        for (int half = 0; half < 2 && 32 * half < nv; ++half) {
          half_tile<NQ>(kaddr + half * (SLOT / 2), v + half * (V_TILE / 2), nv - 32 * half, skip, __int_as_float(lazy), qf, o, st, kept);
        }
        if (--until == 0) lazy = __float_as_int(lazy < 0 ? 0.f : kLazy);   // (bits: minus infinity is the one below zero)
        tally += NQ + ((unsigned)(nv > 32 ? NQ * kept : 2 * NQ * kept) << 16);
        leave(slot);
        // (Only waves that are waiting for a tile ask for tiles: having every wave look for room after each of
        // its tiles cost the busy ones more than the earlier requests saved.)
      }
    }
  };
  // A wave whose second 32 queries are all pad slots (one block in seven on a 30x52 grid) leaves them out.  Measured against
  // working on them: 30x52 with 21 frames, 24 heads 2.87 -> 2.82 ms, 9 frames, 8 heads 380 -> 365 us, matrix instructions 7.53e7
  // -> 7.04e7 and, dense with 3 heads, 6.17e7 -> 5.73e7 (its time, 1.91 ms, stays: other workgroups set it).  One loop for
  // each: as a branch around the tile, in one loop, the two leave the registers in different places and 150 of them go
  // through memory.
  if (two) {
    walk(std::integral_constant<int, 2>());
  } else {
    walk(std::integral_constant<int, 1>());
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[1][dt][i] = nought;    // (not kept through the loop)
  }
  publish();
  if (tile_counts != nullptr && lane == 0 && tally) {
    atomicAdd(&tile_counts[0], (unsigned long long)(tally & 0xffffu));
    // (odd: up in every other wave, whether the waves of a workgroup share lists or not)
    atomicAdd(&tile_counts[1], (unsigned long long)(((tally >> 16) + ((lgroup + part) & 1)) >> 1));
  }
  if (gave_up && lane == 0) {
    atomicAdd(&g_wait_failures, 1ull);
    atomicOr(&ctrl[29], 1 << lgroup);
  }
  __syncthreads();                                    // everyone is done with the ring: reuse it to put the halves together

  lane = opaque_lane();
  const int r = lane & 31, hh = lane >> 5;
  float2* const ml = (float2*)(smem + RING_BYTES) + lane;               // [WAVES][64] reference and normaliser (the bitmaps are done with)
  // ---- where a group has more than two waves: the upper half of them hands over what it has, the lower half adds it to
  // its own, until two are left (four waves hand over 32 KB each at first: the ring's place holds that)
  for (int half = parts >> 1; half >= 2; half >>= 1) {
    unsigned char* const place = smem + ((part & (half - 1)) * groups + lgroup) * (RING_BYTES / 4);
    float2* const pml = ml + ((part & (half - 1)) * groups + lgroup) * 128;
    if (part >= half && part < 2 * half) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
          for (int a = 0; a < 4; ++a)
            *(float4*)(place + (((h * 4 + dt) * 4 + a) * 64 + lane) * 16) =
                make_float4(o[h][dt][4 * a], o[h][dt][4 * a + 1], o[h][dt][4 * a + 2], o[h][dt][4 * a + 3]);
        pml[h * 64] = make_float2(st[h].m, st[h].l);
      }
    }
    __syncthreads();
    if (part < half) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float2 other = pml[h * 64];
        const float m_all = fmaxf(st[h].m, other.x);
        const float a_mine = st[h].m == m_all ? 1.f : __builtin_amdgcn_exp2f((st[h].m - m_all) * kC2);
        const float a_other = other.x == m_all ? 1.f : __builtin_amdgcn_exp2f((other.x - m_all) * kC2);
        st[h].m = m_all;
        st[h].l = st[h].l * a_mine + other.y * a_other;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            const float4 y = *(const float4*)(place + (((h * 4 + dt) * 4 + a) * 64 + lane) * 16);
            o[h][dt][4 * a] = o[h][dt][4 * a] * a_mine + y.x * a_other;
            o[h][dt][4 * a + 1] = o[h][dt][4 * a + 1] * a_mine + y.y * a_other;
            o[h][dt][4 * a + 2] = o[h][dt][4 * a + 2] * a_mine + y.z * a_other;
            o[h][dt][4 * a + 3] = o[h][dt][4 * a + 3] * a_mine + y.w * a_other;
          }
      }
    }
    __syncthreads();
  }

  // ---- the (last) two waves of a group: each hands over what it has of 32 queries and puts the other 32 together
  unsigned char* const given = smem + (part * groups + lgroup) * (RING_BYTES / WAVES);      // 16 KB to hand over in
  unsigned char* const taken = smem + ((part ^ 1) * groups + lgroup) * (RING_BYTES / WAVES);
  auto give = [&](const f32x16 (&x)[4], const Soft& sx) {
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int a = 0; a < 4; ++a)
        *(float4*)(given + ((dt * 4 + a) * 64 + lane) * 16) = make_float4(x[dt][4 * a], x[dt][4 * a + 1], x[dt][4 * a + 2], x[dt][4 * a + 3]);
    ml[(part * groups + lgroup) * 64] = make_float2(sx.m, sum_across_halves(sx.l));
  };
  if (parts > 1) {
    if (part == 0) give(o[1], st[1]);
    else if (part == 1) give(o[0], st[0]);
    __syncthreads();
    if (part > 1) return;                             // (put together with another wave's)
  }
  const bool failed = (ctrl[29] >> lgroup) & 1;        // a wait ran out: say so with NaN rather than with wrong numbers
  unsigned char* const o0 = Op + row_base(q.out);
  // ---- normalise, convert, stage through LDS, write rows of 256 B.  x, sx: 32 queries (number h) of mine, or, with
  // `joined`, what I have of them, the rest being the partner's
  auto finish = [&](int h, const f32x16 (&x)[4], const Soft& sx, auto joined) {
    unsigned char* const turn = joined ? taken : given;
    if (32 * h >= q_valid) {
      // 32 pad slots and nothing else: their rows of the reordered output are zeroed (in the original
      // order they do not exist)
      if (has_block && !direct) {
        const long long row0 = qb * BLOCK + BS * qsub + 32 * h;
#pragma unroll
        for (int it = 0; it < 8; ++it) {
          const int row = it * 4 + (lane >> 4), ch = lane & 15;
          *(uint4*)(Op + (row0 + row) * (D * 2) + ch * 16) = make_uint4(0u, 0u, 0u, 0u);
        }
        if (lse && lane < 32) lse[row0 + lane] = 0.f;
      }
      return;
    }
    const float l_mine = sum_across_halves(sx.l);
    float2 other = make_float2(-FLT_MAX, 0.f);
    if constexpr (joined) other = ml[((part ^ 1) * groups + lgroup) * 64];
    const float m_all = fmaxf(sx.m, other.x);
    const float a_mine = l_mine > 0.f ? __builtin_amdgcn_exp2f((sx.m - m_all) * kC2) : 0.f;
    const float a_other = other.y > 0.f ? __builtin_amdgcn_exp2f((other.x - m_all) * kC2) : 0.f;
    const float lt = l_mine * a_mine + other.y * a_other;
    const float inv = lt > 0.f ? 1.0f / lt : 0.f;     // 0 only in pad query slots whose waves skipped every tile, for an empty list and
    const bool none = lt == 0.f && before > 0 && 32 * h + r < q_valid;   // for keys that all score minus infinity: no softmax is defined, NaN
    if (lse && hh == 0) lse[qb * BLOCK + BS * qsub + 32 * h + r] = m_all * kScale + __logf(lt);
    const float f_mine = a_mine * inv, f_other = a_other * inv;
    uint2 w2[4][4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        // registers 4a..4a+3 are d = 32dt + 8a + 4hh + 0..3 of query r
        float4 y = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (joined) y = *(const float4*)(taken + ((dt * 4 + a) * 64 + lane) * 16);
        f32x2 v0 = {x[dt][4 * a] * f_mine + y.x * f_other, x[dt][4 * a + 1] * f_mine + y.y * f_other};
        f32x2 v1 = {x[dt][4 * a + 2] * f_mine + y.z * f_other, x[dt][4 * a + 3] * f_mine + y.w * f_other};
        bf16x2 b0 = __builtin_convertvector(v0, bf16x2);
        bf16x2 b1 = __builtin_convertvector(v1, bf16x2);
        w2[dt][a] = failed || none ? make_uint2(0x7fc07fc0u, 0x7fc07fc0u) : make_uint2(*(unsigned*)&b0, *(unsigned*)&b1);
      }
    // (all of the partner's share has been read: its place serves to turn the rows)
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int a = 0; a < 4; ++a) *(uint2*)(turn + r * O_STRIDE + (32 * dt + 8 * a + 4 * hh) * 2) = w2[dt][a];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    auto write_rows = [&](auto there) {
#pragma unroll
      for (int it = 0; it < 8; ++it) {
        const int row = it * 4 + (lane >> 4), ch = lane & 15, slot = BS * qsub + 32 * h + row;
        if (!there || slot < rows_there)
          *(uint4*)(o0 + row_after(q.out, slot, there) + ch * 16) = *(const uint4*)(turn + row * O_STRIDE + ch * 16);
      }
    };
    if (direct) write_rows(std::true_type());
    else write_rows(std::false_type());
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  if (parts == 1) {
    finish(0, o[0], st[0], std::false_type());
    finish(1, o[1], st[1], std::false_type());
  } else if (part) {
    finish(1, o[1], st[1], std::true_type());
  } else {
    finish(0, o[0], st[0], std::true_type());
  }
}

}  // namespace ring

// 0: the kernel cannot run this problem, else 1.
int attn_bf16_ring_fits(const Geo& q, bool any_length) {
  if (q.block != ring::BS && q.block != 2 * ring::BS) return 0;
  return ring::lists_fit(q.g, q.k, q.block / ring::BS, any_length);
}

hipError_t launch_attn_bf16_ring(const Geo& q, const void* Qp, const void* Kp, const void* Vt, const int32_t* idx,
                                 const int32_t* row_ptr, long long cap, void* Op, float* lse, bool direct,
                                 unsigned long long* tile_counts, hipStream_t s) {
  const int sub = q.block / ring::BS;
  const int least = ring::least_split(q.g, q.k, sub, row_ptr != nullptr);
  const ring::Share share = ring::share_out((long long)q.B * q.H, (long long)q.g * sub, (long long)q.k * sub, row_ptr != nullptr, least);
  const float skip = log2f((float)q.k * (float)q.block) + ring::kDropLog2;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(share.grid), dim3(512), 0, s, q, (const unsigned char*)Qp, (const unsigned char*)Kp,
                       (const unsigned char*)Vt, idx, row_ptr, cap, (unsigned char*)Op, lse, skip, direct ? 1 : 0,
                       share, tile_counts);
  };
  if (sub == 1 && !row_ptr) go(ring::attn_bf16_ring_kernel<1, false>);
  else if (sub == 1) go(ring::attn_bf16_ring_kernel<1, true>);
  else if (!row_ptr) go(ring::attn_bf16_ring_kernel<2, false>);
  else go(ring::attn_bf16_ring_kernel<2, true>);
  return hipGetLastError();
}

// Waves that gave up waiting for a tile since the library was loaded on the current device (synchronises).
hipError_t read_wait_failures(unsigned long long* count) {
  hipError_t e = hipDeviceSynchronize();
  if (e != hipSuccess) return e;
  return hipMemcpyFromSymbol(count, HIP_SYMBOL(ring::g_wait_failures), sizeof(*count), 0, hipMemcpyDeviceToHost);
}

}  // namespace da
