// Draft logits L = Q~ K~^T / sqrt(d) and the draft attention map softmax(L) (Definition 3.2).
//
// The kept-block decision is taken from these logits, so they are evaluated in float32 with
// one fixed order that a CPU can repeat bit for bit: acc = fma(q[c], k[c], acc) for c ascending
// (the IEEE fused multiply-add: one rounding per term; no split sums), then one multiply by
// float(1/sqrt(d)).  v_mfma_f32_32x32x2_f32 computes exactly that chain: an output is
// fma(a1, b1, fma(a0, b0, c)) with each step rounded once, to nearest even, subnormals kept (its
// results equal fmaf's bit for bit on random, widely scaled, subnormal and overflowing operands,
// and the parity tests hold every logit against the chain).  So the product runs on the matrix
// cores at twice the rate of one fused multiply-add per lane and cycle.
//
// A workgroup of four waves owns a 64x64 tile of L, a wave a 32x32 quarter of it.  Channels come through LDS 32 at a
// time, the next 32 on their way to registers meanwhile; a row is stored with its even channels first and its odd ones
// behind, because lanes 0..31 of an instruction hold channel 2t and lanes 32..63 channel 2t + 1: one 16-byte read then
// serves four instructions.
//
// Measured against an 8x8 piece per thread of a 128x128 tile on the vector ALUs (at its issue rate on large maps, four
// workgroups on small ones): 24 x 1980 x 1980 x 128 channels 295 -> 280 us, 24 x 588 x 588 53 -> 38 us,
// 5 x 1260 x 1260 40 -> 33 us, 48 x 28 x 28 25 -> 5.5 us, 2 x 8 x 8 (64 channels) 13.4 -> 3.7 us.  On the largest the
// products alone take 220 us (110 TFLOP/s; the instruction reaches 130 in a bare loop) and the writing of the map, whose
// rows start anywhere in a cache line, adds the rest.  128x128 tiles measure the same there (282 us), 12 us where 64x64
// take 5; a stretch of consecutive tiles per XCD changes nothing (278 us).
#include <math.h>
#include "da_internal.h"
#include "select_keys.h"

// The compiler contracts nothing in this file (the pragma covers the code below, and the build also
// passes -ffp-contract=off for it): the only fused multiply-adds are the ones written out.
#pragma clang fp contract(off)

namespace da {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int TM = 64;         // tile rows (query blocks) and columns (key blocks) of a workgroup
constexpr int TC = 32;         // channels per LDS stage
constexpr int LDR = TC + 4;    // padded row: the 16-byte reads of 32 rows meet no bank conflict

__global__ __launch_bounds__(256) void draft_logits_kernel(Geo q, const float* __restrict__ q_pool,
                                                           const float* __restrict__ k_pool, float* __restrict__ logits,
                                                           float scale) {
  constexpr int NV = TM * (TC / 4) / 256;              // 16-byte loads of a stage per thread and matrix
  __shared__ __attribute__((aligned(16))) float smem[2 * TM * LDR];
  float* const qs = smem;
  float* const ks = smem + TM * LDR;
  const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const long long bh = blockIdx.z;
  const int row0 = blockIdx.y * TM, col0 = blockIdx.x * TM;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;   // the wave's corner of the tile
  const float* qb = q_pool + bh * (long long)q.g * q.d;
  const float* kb = k_pool + bh * (long long)q.g * q.d;
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;

  // loader: load v of thread tid is channels 4 (tid % 8) .. +3 of row tid / 8 + 32 v.  No load sits behind a branch:
  // what lies past the last row or channel reads the last one and is not used (d is a multiple of 4).
  const int lr = tid >> 3, lc = 4 * (tid & 7);
  f32x4 nq[NV], nk[NV];
  auto fetch = [&](int c0) {
    const int c = min(c0 + lc, q.d - 4);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      nq[v] = *(const f32x4*)(qb + (long long)min(row0 + lr + 32 * v, q.g - 1) * q.d + c);
      nk[v] = *(const f32x4*)(kb + (long long)min(col0 + lr + 32 * v, q.g - 1) * q.d + c);
    }
  };
  // eight channels (or, `half`, the first four of them) of the stage
  auto eight = [&](int u, bool half) {
    const float4 a = *(const float4*)&qs[(wr + r32) * LDR + hh * (TC / 2) + 4 * u];
    const float4 b = *(const float4*)&ks[(wc + r32) * LDR + hh * (TC / 2) + 4 * u];
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, acc, 0, 0, 0);
    if (half) return;
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, acc, 0, 0, 0);
  };
  const bool works = row0 + wr < q.g && col0 + wc < q.g;   // else all of the wave's tile lies outside
  auto stage = [&]() {
    __syncthreads();                                     // everyone has left the previous stage
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      // (the loads are waited for here and not, for the sake of the shuffle below, where they are asked for)
      asm volatile("" : "+v"(nq[v]), "+v"(nk[v]));
      float* const qd = qs + (lr + 32 * v) * LDR + lc / 2;
      float* const kd = ks + (lr + 32 * v) * LDR + lc / 2;
      *(float2*)qd = make_float2(nq[v].x, nq[v].z);
      *(float2*)(qd + TC / 2) = make_float2(nq[v].y, nq[v].w);
      *(float2*)kd = make_float2(nk[v].x, nk[v].z);
      *(float2*)(kd + TC / 2) = make_float2(nk[v].y, nk[v].w);
    }
    __syncthreads();
  };
  fetch(0);
  int c0 = 0;
  for (; c0 + TC <= q.d; c0 += TC) {
    stage();
    fetch(c0 + TC);                                      // (past the end: the last channels again, not used)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < TC / 8; ++u) eight(u, false);
  }
  if (c0 < q.d) {
    stage();
    for (int c = c0; c < q.d; c += 8) eight((c - c0) >> 3, c + 4 >= q.d);
  }
  // Accumulator register r of lane l: row 8(r/4) + 4(l/32) + r%4, column l%32 of the wave's 32x32 piece.  It goes out by
  // way of LDS (each wave through a stretch of its own), 16 bytes per lane and 128 bytes of a row in one piece.
  __syncthreads();                                       // the last stage has been read
  if (!works) return;
  float* out = logits + bh * (long long)q.g * q.g;
  float* const mine = smem + wave * 32 * LDR;            // (4 * 32 rows of LDR floats: exactly smem)
#pragma unroll
  for (int r = 0; r < 16; ++r) mine[(8 * (r >> 2) + 4 * hh + (r & 3)) * LDR + r32] = acc[r] * scale;
  __builtin_amdgcn_wave_barrier();
  const int rw = row0 + wr, cw = col0 + wc;
  if ((q.g & 3) == 0) {
    // g a multiple of 4: four columns are inside the row or outside it as a whole, and 16-byte aligned
#pragma unroll
    for (int e0 = 0; e0 < 32 * 8; e0 += 64) {
      const int e = e0 + lane, r = e >> 3, c = 4 * (e & 7);
      const float4 v = *(const float4*)&mine[r * LDR + c];
      if (rw + r < q.g && cw + c < q.g) *(float4*)(out + (long long)(rw + r) * q.g + cw + c) = v;
    }
  } else {
    for (int e = lane; e < 32 * 32; e += 64) {
      const int r = e >> 5, c = e & 31;
      const float v = mine[r * LDR + c];
      if (rw + r < q.g && cw + c < q.g) out[(long long)(rw + r) * q.g + cw + c] = v;
    }
  }
}

// Logits and lists in one launch where a row of the map is short (g <= kFusedColumns): a workgroup of eight waves owns 32
// rows of one head's map, a wave 32 columns of them, and the map goes no further than LDS.  Small launches do not
// fill the chip, and what they take is a chain of latencies: one launch less, no trip of the map through memory, and the
// operands come straight from the pooled rows into registers, without stages and barriers (a lane asks for four channels at
// a time and uses the two of its half-wave: the chain of products is draft_logits_kernel's, and so are the bits).
// The lists follow select_reg_kernel: a wave takes four rows, side by side, so that a bit costs one latency and not four.
// da_forward, us, two launches -> one: 2 x 8 x 8 (64 channels) 23.7 -> 21.7, 2 x 25 x 25 49.1 -> 46.4, 48 x 28 x 28 104.6 ->
// 102.6.  Wider rows gain nothing (4 x 84 x 84 193 either way) or lose (6 x 180 x 180 145 -> 154, 4 x 240 x 240 431 -> 442; with the
// operands by way of LDS 2 x 252 x 252 120 -> 126): fewer workgroups share the selection, which is then the longer part.
// More than two workgroups for every CU, and the waves without columns or rows cost more than the launch, unless most of a tile's 32
// rows are there (maps x g x g, da_forward, two launches / one, what is taken in *): 384 x 3 73.6 / *72.9*, x 8 118.5 / *116.8*, x 12 197.3 /
// *196.5*, 192 x 40 260.8 / *257.5*, 288 x 40 *382* / 384, 576 x 40 *763* / 768, x 64 *1605* / 1602, 768 x 4 *122.9* / 124.4, 1536 x 4 *242* / 257, x 9 *657* /
// 668, but 384 x 16 254.7 / *251.8*, x 28 615.9 / *611.8*, 1536 x 28 2374 / *2360*, x 32 2756 / *2733*.
constexpr int kFusedColumns = 64;
constexpr int FR = 32;                                   // rows of a workgroup
constexpr int FW = 8;                                    // waves
constexpr int FS = FR / FW;                              // rows per wave of the selection

__global__ __launch_bounds__(64 * FW) void draft_select_kernel(Geo q, const float* __restrict__ q_pool,
                                                               const float* __restrict__ k_pool, int32_t* __restrict__ idx,
                                                               float scale, int row_tiles) {
  constexpr int LDM = kFusedColumns + 4;
  __shared__ float map[FR * LDM];
  const int lane = threadIdx.x & 63, r32 = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bh = (int)(blockIdx.x / (unsigned)row_tiles);
  const int row0 = ((int)blockIdx.x - bh * row_tiles) * FR, col0 = wave * 32;
  if (col0 < q.g) {
    // (rows past the last one read that again and are not used)
    const float* const qr = q_pool + ((long long)bh * q.g + min(row0 + r32, q.g - 1)) * q.d;
    const float* const kr = k_pool + ((long long)bh * q.g + min(col0 + r32, q.g - 1)) * q.d;
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    constexpr int CH = 64;                               // channels asked for at a time
    for (int c0 = 0; c0 < q.d; c0 += CH) {               // (d is 64 or 128 here)
      f32x4 a[CH / 4], b[CH / 4];
#pragma unroll
      for (int u = 0; u < CH / 4; ++u) {
        a[u] = *(const f32x4*)(qr + c0 + 4 * u);
        b[u] = *(const f32x4*)(kr + c0 + 4 * u);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < CH / 4; ++u) {
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(hh ? a[u].y : a[u].x, hh ? b[u].y : b[u].x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(hh ? a[u].w : a[u].z, hh ? b[u].w : b[u].z, acc, 0, 0, 0);
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) map[(8 * (r >> 2) + 4 * hh + (r & 3)) * LDM + col0 + r32] = acc[r] * scale;
  }
  __syncthreads();
  const int g = q.g, k = q.k;
  unsigned key[FS];                                      // of column `lane`
#pragma unroll
  for (int w = 0; w < FS; ++w) key[w] = lane < g ? order_key(map[(wave * FS + w) * LDM + lane]) : 0u;
  // the value that k keys reach, bit by bit from the top; a row at whose value exactly k keys arrive is done
  unsigned thr[FS];
  bool cut[FS];
#pragma unroll
  for (int w = 0; w < FS; ++w) thr[w] = 0u, cut[w] = false;
  for (int bit = 31; bit >= 0; --bit) {
    bool all = true;
#pragma unroll
    for (int w = 0; w < FS; ++w) {
      const unsigned cand = thr[w] | (1u << bit);
      const int cnt = __popcll(__ballot(key[w] >= cand));
      if (!cut[w] && cnt >= k) thr[w] = cand;
      cut[w] = cut[w] || cnt == k;
      all = all && cut[w];
    }
    if (all) break;                                      // (the same in every lane)
  }
#pragma unroll
  for (int w = 0; w < FS; ++w) {
    const int row = row0 + wave * FS + w;
    if (row >= g) break;                                 // (the same in every lane)
    // what beats the value, and of what equals it the first columns, as many as are still wanted (cut: k keys reach the value,
    // so all that equal it are)
    const unsigned long long gt_mask = __ballot(key[w] > thr[w]), eq_mask = __ballot(lane < g && key[w] == thr[w]);
    const bool take = (gt_mask >> lane & 1) || ((eq_mask >> lane & 1) && lane_prefix(eq_mask) < k - __popcll(gt_mask));
    const unsigned long long take_mask = __ballot(take);
    if (take) idx[((long long)bh * g + row) * k + lane_prefix(take_mask)] = lane;
  }
}

__device__ inline float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}
__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// One wavefront per row; safe in place (every element is read before it is written by the
// same lane, and rows do not overlap).
__global__ __launch_bounds__(256) void row_softmax_kernel(const float* logits, float* draft, int g, long long rows) {
  long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  int lane = threadIdx.x & 63;
  const float* in = logits + row * g;
  float* out = draft + row * g;
  float m = -INFINITY;
  for (int j = lane; j < g; j += 64) m = fmaxf(m, in[j]);
  m = wave_max(m);
  float z = 0.f;
  for (int j = lane; j < g; j += 64) z += expf(in[j] - m);
  z = wave_sum(z);
  float inv = 1.0f / z;
  for (int j = lane; j < g; j += 64) out[j] = expf(in[j] - m) * inv;
}

hipError_t launch_draft_logits(const Geo& q, const float* q_pool, const float* k_pool, float* logits, hipStream_t s) {
  const float scale = (float)(1.0 / sqrt((double)q.d));
  const long long bh = (long long)q.B * q.H;
  const unsigned t = (unsigned)((q.g + TM - 1) / TM);
  hipLaunchKernelGGL(draft_logits_kernel, dim3(t, t, (unsigned)bh), dim3(256), 0, s, q, q_pool, k_pool, logits, scale);
  return hipGetLastError();
}

hipError_t launch_row_softmax(const Geo& q, const float* logits, float* draft, hipStream_t s) {
  long long rows = (long long)q.B * q.H * q.g;
  hipLaunchKernelGGL(row_softmax_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, logits, draft, q.g, rows);
  return hipGetLastError();
}

bool draft_select_fits(const Geo& q) {
  const long long groups = (q.g + FR - 1) / FR * (long long)q.B * q.H;
  return q.g <= kFusedColumns && q.d % 64 == 0 && (groups <= 512 || (q.g >= FR / 2 && q.g <= FR));
}

hipError_t launch_draft_select(const Geo& q, const float* q_pool, const float* k_pool, int32_t* idx, hipStream_t s) {
  const float scale = (float)(1.0 / sqrt((double)q.d));
  const int row_tiles = (q.g + FR - 1) / FR;
  hipLaunchKernelGGL(draft_select_kernel, dim3((unsigned)(row_tiles * (long long)q.B * q.H)), dim3(64 * FW), 0, s, q, q_pool, k_pool,
                     idx, scale, row_tiles);
  return hipGetLastError();
}

}  // namespace da
