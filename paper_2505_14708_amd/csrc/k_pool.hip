// Average pooling of Q and K inside each latent frame (Definition 3.2); with MAXP the maximum instead
// (the other downsampling kernel of the ablation, Section 4.3).
// HBM-bound: Q and K are read once in 16-byte pieces straight from the original layout
// (the tokens of a patch row are contiguous); each lane owns a fixed group of channels of
// one block and adds the block's tokens in slot order, so the float32 result does not
// depend on the launch shape:  acc = acc + x (one rounding per add), mean = acc / valid.
// Q and K are read once and never again by this pass: the loads are marked non-temporal, so the stream does not
// push anything else out of the L2 (measured on the headline shape: 5.4 -> 5.8 TB/s).
#include <type_traits>
#include "da_internal.h"
#include "vt_block.h"

#pragma clang fp contract(off)

namespace da {

template <int DT>
struct Vec;
template <>
struct Vec<DA_BF16> {
  static constexpr int N = 8;
  __device__ static void widen(const uint4& r, float* f) {
    const unsigned w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f[2 * j] = __uint_as_float(w[j] << 16);
      f[2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u);
    }
  }
};
template <>
struct Vec<DA_F32> {
  static constexpr int N = 4;
  __device__ static void widen(const uint4& r, float* f) {
    f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y);
    f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
  }
};

constexpr int kPoolThreads = 64;

// Item number `item` of the (bh, block, chunk) of X.  With Kp (X is then K) the tokens are also written, as they go by,
// to their slots of the reordered tensor Kp (Algorithm 1), pad slots zeroed: pooling and reordering then
// read K once between them.
template <int DT, bool MAXP>
__device__ __forceinline__ void pool_item(const Geo& q, const uint4* __restrict__ X, float* __restrict__ out,
                                          uint4* __restrict__ Kp, int cpr, long long item) {
  constexpr int N = Vec<DT>::N;
  long long blk = item / cpr;  // over bh * g
  int c = (int)(item - blk * cpr);
  long long bh = blk / q.g;
  int i = (int)(blk - bh * q.g);
  BlockPos b = block_pos(q, i);
  // chunks between consecutive rows of the source, rows between the block's patch rows
  const long long sn = q.in.sn / N;
  const long long pitch = block_row_pitch(q, b);
  const uint4* src = X + row_offset(q.in, q.H, bh, block_first_row(q, i, b)) / N + c;
  const bool wr = Kp != nullptr;
  uint4* dstp = wr ? Kp + (blk * q.block) * cpr + c : nullptr;   // slot 0 of the block
  float acc[N];
#pragma unroll
  for (int j = 0; j < N; ++j) acc[j] = MAXP ? -INFINITY : 0.f;
  // one token's channels go into the running sum, or (MAXP) replace the running maximum where larger
  auto take = [&](const float (&f)[N]) {
#pragma unroll
    for (int j = 0; j < N; ++j) acc[j] = MAXP ? (f[j] > acc[j] ? f[j] : acc[j]) : acc[j] + f[j];
  };
  int u = 0;
  // two full patch rows at a time where the patch is 8 wide: sixteen independent loads in flight,
  // added in slot order
  if (b.vw == 8) {
    for (; u + 2 <= b.vh; u += 2) {
      const uint4* row = src + (long long)u * pitch * sn;
      uint4 r[16];
#pragma unroll
      for (int t = 0; t < 16; ++t) r[t] = load_once(&row[((long long)(t >> 3) * pitch + (t & 7)) * sn]);
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        if (wr) dstp[(long long)(u * 8 + t) * cpr] = r[t];
        float f[N];
        Vec<DT>::widen(r[t], f);
        take(f);
      }
    }
  }
  for (; u < b.vh; ++u) {
    const uint4* row = src + (long long)u * pitch * sn;
    int v = 0;
    for (; v + 8 <= b.vw; v += 8) {  // eight independent loads in flight, added in order
      uint4 r[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) r[t] = load_once(&row[(long long)(v + t) * sn]);
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        if (wr) dstp[(long long)(u * b.vw + v + t) * cpr] = r[t];
        float f[N];
        Vec<DT>::widen(r[t], f);
        take(f);
      }
    }
    for (; v < b.vw; ++v) {
      const uint4 rv = load_once(&row[(long long)v * sn]);
      if (wr) dstp[(long long)(u * b.vw + v) * cpr] = rv;
      float f[N];
      Vec<DT>::widen(rv, f);
      take(f);
    }
  }
  if (wr)
    for (int sl = b.vh * b.vw; sl < q.block; ++sl) dstp[(long long)sl * cpr] = make_uint4(0u, 0u, 0u, 0u);
  float cnt = (float)(b.vh * b.vw);
  float* dst = out + blk * q.d + c * N;
#pragma unroll
  for (int j = 0; j < N; ++j) dst[j] = MAXP ? acc[j] : acc[j] / cnt;   // IEEE division (correctly rounded is the compiler default for HIP)
}

// The same for launches that are too small to fill the chip (kSmallWaves) on grids that leave patch rows of fewer than
// eight tokens: there a wave's turns at memory, one after the other, are the time, not the bytes, and pool_kernel takes
// up to 64 of them where a patch row is cut (one token at a time; four where all are eight wide).  Here a lane owns 8
// bytes of a block's rows instead of 16, which makes twice as many waves, and the loads of 64 tokens are all on their
// way before the first is used, whatever the block's extent (slots past the last valid one read that again).  The order
// of the sums is the same, token by token.  da_forward, one 30x52 frame, 48 heads: 109 -> 91 us; three of them in
// float32, 4 heads: 115 -> 107 us; where every patch is eight wide (48x80, 24 heads) 109 us either way and on the
// smallest 21.4 -> 22.5 us, so those stay with pool_kernel.
template <int DT, bool MAXP>
__device__ __forceinline__ void pool_small_item(const Geo& q, const uint2* __restrict__ X, float* __restrict__ out,
                                                uint2* __restrict__ Kp, int cpr, unsigned item) {
  constexpr int N = Vec<DT>::N / 2;
  constexpr int AHEAD = 64;
  // (few: 32 bits hold their numbers, and 64-bit divisions are five times as long)
  const unsigned in_head = item / (unsigned)cpr;   // over bh * g
  const int c = (int)(item - in_head * (unsigned)cpr);
  const long long blk = in_head, bh = in_head / (unsigned)q.g;
  const int i = (int)(in_head - (unsigned)bh * (unsigned)q.g);
  const BlockPos b = block_pos(q, i);
  const int nv = b.vh * b.vw;
  const unsigned sn = (unsigned)(q.in.sn / N);                            // pieces between consecutive rows of the source (the launcher has seen that it fits)
  const int skip = block_row_pitch(q, b) - b.vw;                          // rows between a patch row's last token and the next one's first
  const int recip = (65536 + b.vw - 1) / b.vw;                            // slot / vw by way of the reciprocal: exact below 256
  const uint2* src = X + row_offset(q.in, q.H, bh, block_first_row(q, i, b)) / N + c;
  const bool wr = Kp != nullptr;
  uint2* dstp = wr ? Kp + (blk * q.block) * cpr + c : nullptr;   // slot 0 of the block
  float acc[N];
#pragma unroll
  for (int j = 0; j < N; ++j) acc[j] = MAXP ? -INFINITY : 0.f;
  for (int s0 = 0; s0 < nv; s0 += AHEAD) {
    uint2 r[AHEAD];
#pragma unroll
    for (int t = 0; t < AHEAD; ++t) {
      const int s = min(s0 + t, nv - 1);
      r[t] = src[(unsigned long long)(unsigned)(((s * recip) >> 16) * skip + s) * sn];
    }
#pragma unroll
    for (int t = 0; t < AHEAD; ++t) {
      const bool in = s0 + t < nv;
      if (wr && s0 + t < q.block) dstp[(long long)(s0 + t) * cpr] = in ? r[t] : make_uint2(0u, 0u);
      float f[Vec<DT>::N];
      Vec<DT>::widen(make_uint4(r[t].x, r[t].y, 0u, 0u), f);
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const float with = MAXP ? (f[j] > acc[j] ? f[j] : acc[j]) : acc[j] + f[j];
        acc[j] = in ? with : acc[j];
      }
    }
  }
  if (wr)
    for (int sl = (nv + AHEAD - 1) / AHEAD * AHEAD; sl < q.block; ++sl) dstp[(long long)sl * cpr] = make_uint2(0u, 0u);
  const float cnt = (float)nv;
  float* dst = out + blk * q.d + c * N;
#pragma unroll
  for (int j = 0; j < N; ++j) dst[j] = MAXP ? acc[j] : acc[j] / cnt;
}

// grid.x covers the items; grid.y = 0 for Q, 1 for K
template <int DT, bool SMALL, bool MAXP>
__global__ __launch_bounds__(kPoolThreads, SMALL ? 2 : 1) void pool_kernel(Geo q, const void* __restrict__ Q,
                                                                           const void* __restrict__ K, float* __restrict__ q_pool,
                                                                           float* __restrict__ k_pool, int cpr, long long items) {
  const long long item = (long long)blockIdx.x * kPoolThreads + threadIdx.x;
  if (item >= items) return;
  const void* const X = blockIdx.y ? K : Q;
  float* const out = blockIdx.y ? k_pool : q_pool;
  if constexpr (SMALL) pool_small_item<DT, MAXP>(q, (const uint2*)X, out, nullptr, cpr, (unsigned)item);
  else pool_item<DT, MAXP>(q, (const uint4*)X, out, nullptr, cpr, item);
}

// What stands before the draft logits and the attention, in one launch: pooling of Q, pooling of K with its reordering,
// and the reordering of V as operands.  They have nothing to do with each other, so where a launch of one does not fill the chip
// the others do; where it does, a tail and a launch are saved.  `per` workgroups for Q, as many for K, then one per block of V (the
// shorter ones last).
// da_forward, us, two launches -> one: 2 x 28 blocks 42.6 -> 39.2, 48 x 28 102.6 -> 97.1, 24 x 60 (48x80) 117.7 -> 114.8, 24 x 252
// 922 -> 906, 8 x 540 1320 -> 1302, 30 x 63 (one of 47x39) 764 -> 741.
// With K in block order already (no Kp), short launches gain as much (2 x 28 blocks 38.6 -> 37.1, 8 x 60 63.2 -> 59.8), longer ones lose
// (24 x 84 162 -> 165, 76 x 84 222 -> 228, 8 x 392 711 -> 717): the two streams of reads run better one after the other there.
// The line, kInPlaceBlocks, lies where it makes no difference (36 x 28 71.0 and 71.6).
// Where each of the three fills the chip by itself there is little in it: 24 x 720 blocks 2.42 and 2.43 ms, 24 x 1260 6.42 and 6.41, 24 x 1980 15.41
// and 15.37, 12 x 3900 29.97 and 29.90, 24 x 990 of 128 slots 11.58 and 11.58 (the launch itself 657 us against 650 for the two at 24 x 1980).
constexpr int kPrepThreads = 256;
template <bool SMALL, bool MAXP>
__global__ __launch_bounds__(kPrepThreads, SMALL ? 2 : 1) void prepare_kernel(Geo q, const void* __restrict__ Q,
                                                                              const void* __restrict__ K,
                                                                              const uint16_t* __restrict__ V,
                                                                              float* __restrict__ q_pool, float* __restrict__ k_pool,
                                                                              void* __restrict__ Kp, uint16_t* __restrict__ Vt,
                                                                              int cpr, long long items, unsigned per) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if (blockIdx.x >= 2 * per) {
    const unsigned b = blockIdx.x - 2 * per, bh = b / (unsigned)q.g;
    vt_block<uint16_t, true>(q, V, Vt, (int)(b - bh * (unsigned)q.g), bh, smem);
    return;
  }
  const bool is_k = blockIdx.x >= per;
  const long long item = (long long)(is_k ? blockIdx.x - per : blockIdx.x) * kPrepThreads + threadIdx.x;
  if (item >= items) return;
  const void* const X = is_k ? K : Q;
  float* const out = is_k ? k_pool : q_pool;
  if constexpr (SMALL) pool_small_item<DA_BF16, MAXP>(q, (const uint2*)X, out, is_k ? (uint2*)Kp : nullptr, cpr, (unsigned)item);
  else pool_item<DA_BF16, MAXP>(q, (const uint4*)X, out, is_k ? (uint4*)Kp : nullptr, cpr, item);
}

// Below this many waves of pool_item in all pool_small_item is taken.  (1008 waves 243 -> 225 us, 2016 waves 391 -> 386 us,
// from 2940 on no difference either way.)
constexpr long long kSmallWaves = 2048;

namespace {
struct Items {
  bool small;
  int cpr;            // items per block
  long long count;
};
Items pool_items(const Geo& q) {
  const int cpr = (int)(q.d * (q.dtype == DA_BF16 ? 2 : 4) / 16);
  const long long items = (long long)q.B * q.H * q.g * cpr;
  const bool cut = q.fw % q.pw != 0 || q.pw % 8 != 0;   // some patch rows are not a multiple of eight tokens
  const bool small = cut && 2 * items < 64 * kSmallWaves && q.block >= 64 && q.block <= 128 && q.in.sn < (1LL << 31);
  return {small, small ? 2 * cpr : cpr, small ? 2 * items : items};
}
// go(small, max) with the two as types
template <typename F>
void pick_pool(const Geo& q, bool small, F go) {
  const std::true_type yes;
  const std::false_type no;
  const bool max_pool = q.pool == DA_POOL_MAX;
  if (small && max_pool) go(yes, yes);
  else if (small) go(yes, no);
  else if (max_pool) go(no, yes);
  else go(no, no);
}
}  // namespace

hipError_t launch_pool(const Geo& q, const void* Q, const void* K, float* q_pool, float* k_pool, hipStream_t s) {
  const Items it = pool_items(q);
  pick_pool(q, it.small, [&](auto small, auto max_pool) {
    constexpr bool SM = decltype(small)::value, MX = decltype(max_pool)::value;
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)((it.count + kPoolThreads - 1) / kPoolThreads), 2), dim3(kPoolThreads), 0, s, q, Q,
                         K, q_pool, k_pool, it.cpr, it.count);
    };
    if (q.dtype == DA_BF16) go(pool_kernel<DA_BF16, SM, MX>);
    else go(pool_kernel<DA_F32, SM, MX>);
  });
  return hipGetLastError();
}

constexpr long long kInPlaceBlocks = 1024;

hipError_t launch_prepare(const Geo& q, const void* Q, const void* K, const void* V, float* q_pool, float* k_pool, void* Kp,
                          void* Vt, hipStream_t s) {
  if (!Kp && (long long)q.B * q.H * q.g >= kInPlaceBlocks) {
    const hipError_t e = launch_pool(q, Q, K, q_pool, k_pool, s);
    return e != hipSuccess ? e : launch_permute(q, V, Vt, DA_REORDER_VOP, s);
  }
  const Items it = pool_items(q);
  const unsigned per = (unsigned)((it.count + kPrepThreads - 1) / kPrepThreads);
  const dim3 grid((unsigned)(2 * per + (long long)q.B * q.H * q.g));
  pick_pool(q, it.small, [&](auto small, auto max_pool) {
    constexpr bool SM = decltype(small)::value, MX = decltype(max_pool)::value;
    hipLaunchKernelGGL((prepare_kernel<SM, MX>), grid, dim3(kPrepThreads), vt_block_lds(q), s, q, Q, K, (const uint16_t*)V, q_pool,
                       k_pool, Kp, (uint16_t*)Vt, it.cpr, it.count, per);
  });
  return hipGetLastError();
}

}  // namespace da
