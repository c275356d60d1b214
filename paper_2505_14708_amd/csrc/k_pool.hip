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

#pragma clang fp contract(off)

namespace da {

// 16 bytes, read once
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ inline uint4 load_once(const uint4* p) {
  const u32x4 v = __builtin_nontemporal_load((const u32x4*)p);
  return make_uint4(v.x, v.y, v.z, v.w);
}

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

// grid.x covers (bh, block, chunk) items; grid.y = 0 for Q, 1 for K.  With REORDER the tokens of K are
// also written, as they go by, to their slots of the reordered tensor Kp (Algorithm 1), pad
// slots zeroed: pooling and reordering then read K once between them.
template <int DT, bool REORDER, bool MAXP>
__global__ __launch_bounds__(kPoolThreads) void pool_kernel(Geo q, const uint4* __restrict__ Q, const uint4* __restrict__ K,
                                                   float* __restrict__ q_pool, float* __restrict__ k_pool,
                                                   uint4* __restrict__ Kp, int cpr, long long items) {
  constexpr int N = Vec<DT>::N;
  long long item = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (item >= items) return;
  const uint4* X = blockIdx.y ? K : Q;
  float* out = blockIdx.y ? k_pool : q_pool;
  long long blk = item / cpr;  // over bh * g
  int c = (int)(item - blk * cpr);
  long long bh = blk / q.g;
  int i = (int)(blk - bh * q.g);
  BlockPos b = block_pos(q, i);
  // chunks between consecutive rows of the source, rows between the block's patch rows
  const long long sn = q.in.sn / N;
  const long long pitch = block_row_pitch(q, b);
  const uint4* src = X + row_offset(q.in, q.H, bh, block_first_row(q, i, b)) / N + c;
  const bool wr = REORDER && blockIdx.y;               // (Q is only pooled)
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
template <int DT, bool REORDER, bool MAXP>
__global__ __launch_bounds__(kPoolThreads, 2) void pool_small_kernel(Geo q, const uint2* __restrict__ Q, const uint2* __restrict__ K,
                                                                     float* __restrict__ q_pool, float* __restrict__ k_pool,
                                                                     uint2* __restrict__ Kp, int cpr, long long items) {
  constexpr int N = Vec<DT>::N / 2;
  constexpr int AHEAD = 64;
  const unsigned item = blockIdx.x * kPoolThreads + threadIdx.x;   // (few: 32 bits hold them, and 64-bit divisions are five times as long)
  if (item >= items) return;
  const uint2* X = blockIdx.y ? K : Q;
  float* out = blockIdx.y ? k_pool : q_pool;
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
  const bool wr = REORDER && blockIdx.y;               // (Q is only pooled)
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

// Below this many waves of pool_kernel in all.  (1008 waves 243 -> 225 us, 2016 waves 391 -> 386 us, from 2940 on no
// difference either way.)
constexpr long long kSmallWaves = 2048;

hipError_t launch_pool(const Geo& q, const void* Q, const void* K, float* q_pool, float* k_pool, hipStream_t s) {
  return launch_pool_reorder(q, Q, K, q_pool, k_pool, nullptr, s);
}

// Kp may be NULL (K is then only pooled); given, dtype is DA_BF16
hipError_t launch_pool_reorder(const Geo& q, const void* Q, const void* K, float* q_pool, float* k_pool, void* Kp,
                               hipStream_t s) {
  size_t es = q.dtype == DA_BF16 ? 2 : 4;
  int cpr = (int)(q.d * es / 16);
  long long items = (long long)q.B * q.H * q.g * cpr;
  const bool cut = q.fw % q.pw != 0 || q.pw % 8 != 0;   // some patch rows are not a multiple of eight tokens
  const bool small = cut && 2 * items < 64 * kSmallWaves && q.block >= 64 && q.block <= 128 && q.in.sn < (1LL << 31);
  auto pick = [&](auto dt, auto reorder, auto max_pool) {
    constexpr int DT = decltype(dt)::value;
    constexpr bool RE = decltype(reorder)::value, MX = decltype(max_pool)::value;
    if (small)
      hipLaunchKernelGGL((pool_small_kernel<DT, RE, MX>), dim3((unsigned)((2 * items + kPoolThreads - 1) / kPoolThreads), 2),
                         dim3(kPoolThreads), 0, s, q, (const uint2*)Q, (const uint2*)K, q_pool, k_pool, (uint2*)Kp, 2 * cpr,
                         2 * items);
    else
      hipLaunchKernelGGL((pool_kernel<DT, RE, MX>), dim3((unsigned)((items + kPoolThreads - 1) / kPoolThreads), 2),
                         dim3(kPoolThreads), 0, s, q, (const uint4*)Q, (const uint4*)K, q_pool, k_pool, (uint4*)Kp, cpr, items);
  };
  auto pick_max = [&](auto dt, auto reorder) {
    if (q.pool == DA_POOL_MAX) pick(dt, reorder, std::true_type());
    else pick(dt, reorder, std::false_type());
  };
  const std::integral_constant<int, DA_BF16> bf16;
  const std::integral_constant<int, DA_F32> f32;
  if (q.dtype != DA_BF16) pick_max(f32, std::false_type());
  else if (Kp) pick_max(bf16, std::true_type());
  else pick_max(bf16, std::false_type());
  return hipGetLastError();
}

}  // namespace da
