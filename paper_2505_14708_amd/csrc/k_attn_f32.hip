// SparseAttn for float32 storage, blocks of 64 slots, d = 64 or 128: float32 throughout, on the float32 matrix
// instructions (v_mfma_f32_32x32x2_f32: exact products, one rounding per term, like a chain of fused multiply-adds).
//
// A workgroup is one query block; its four waves are two halves of the queries times two halves of every key tile, so
// a wave works on 32 queries x 32 keys per tile.  The query is on the lane axis of both products:
//     S^T = K Q^T      lane l: query l % 32; accumulator register r: key 8(r/4) + 4(l/32) + r%4 of the wave's half
//     O^T += V^T P^T   register r of P is, as it stands, the operand of the step that adds the keys 8(r/4) + r%4 (lanes
//                      0..31) and that plus 4 (lanes 32..63): no exchange between lanes
// Channels are taken in whatever order makes the LDS reads wide: a step of the first product pairs channel 8u + j with
// 8u + 4 + j (one 16-byte read of K serves four steps), and row i of accumulator dt of the second product is channel
// (d/32) i + dt (one read of V serves the d/32 accumulators).  The two key halves keep a running maximum, a sum and an
// output of their own and are put together at the end.
//
// What bounds it: the matrix instructions (64 cycles each; a 64 x 64 tile at d = 128 is 8192 cycles of every SIMD
// against 64 KB brought in, 8 bytes per cycle and CU).  The next tile's rows are on their way to registers while the
// present tile is multiplied; LDS holds one tile (66 KB at d = 128), so two workgroups share a CU and one multiplies
// while the other is at its barriers.  Measured against one wave per query block on the vector ALUs with its own tile in
// LDS: 3236 -> 227 us at 84 blocks x 4 heads, d = 128, 21 blocks kept (65 TFLOP/s of the 130 a bare loop of these
// instructions reaches), 134 -> 18 us at 8 blocks x 2 heads, d = 64, 4 kept.
#include <math.h>
#include "da_internal.h"

namespace da {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float across_halves_max(float x) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float across_halves_sum(float x) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// VT: V comes block-transposed (DA_REORDER_VT); otherwise K and V alike are rows that q.in says where to find.
template <int D, bool VT>
__global__ __launch_bounds__(256, 2) void attn_f32_kernel(Geo q, const float* __restrict__ Q, const float* __restrict__ K,
                                                          const float* __restrict__ V, const int32_t* __restrict__ idx,
                                                          const int32_t* __restrict__ row_ptr, long long cap,
                                                          float* __restrict__ O, float* __restrict__ lse) {
  constexpr int LD = D + 4;                  // padded row of a tile in LDS: the 16-byte reads of 32 rows meet no conflict
  constexpr int CPR = D / 4;                 // 16-byte chunks per row
  constexpr int NCH = 64 * CPR / 256;        // chunks of a tile per thread
  constexpr int NDT = D / 32;                // accumulators of the second product
  __shared__ __attribute__((aligned(16))) float ks[64 * LD];
  __shared__ __attribute__((aligned(16))) float vs[64 * LD];
  // workgroups are dealt round-robin to the 8 XCDs: each gets a stretch of consecutive query blocks, whose lists have
  // much in common
  const long long total = (long long)q.B * q.H * q.g, chunk = (total + 7) >> 3;
  const long long qb = (blockIdx.x & 7) * chunk + (blockIdx.x >> 3);
  if ((blockIdx.x >> 3) >= chunk || qb >= total) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qh = wave & 1, kh = wave >> 1;
  const int r32 = lane & 31, hh = lane >> 5;
  const long long bh = qb / q.g;
  const int i_blk = (int)(qb - bh * q.g);
  const float scale_log2 = (float)(1.4426950408889634 / sqrt((double)D));

  // the wave's query row (slots past the valid ones exist only where the tensors are in block order)
  const BlockPos qp = block_pos(q, i_blk);
  const int q_valid = qp.vh * qp.vw, my_slot = 32 * qh + r32;
  const bool has_row = my_slot < q_valid || q.reordered;
  const bool live = 32 * qh < q_valid || q.reordered;        // (the same in every lane)
  const long long q_first = block_first_row(q, i_blk, qp);
  const long long my_row = q_first + (long long)(my_slot / qp.vw) * block_row_pitch(q, qp) + my_slot % qp.vw;
  float4 qv[D / 8];
  {
    const float* qrow = Q + row_offset(q.in, q.H, bh, has_row ? my_row : q_first) + 4 * hh;
#pragma unroll
    for (int u = 0; u < D / 8; ++u) qv[u] = *(const float4*)(qrow + 8 * u);
  }
  f32x16 o[NDT];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[dt][i] = 0.f;
  float m = -INFINITY, l = 0.f;

  // k columns per row, or (row_ptr given) lists of any length, one after the other per head
  const int32_t* list = idx + qb * q.k;
  int len = q.k;
  if (row_ptr) {
    const int32_t* rp = row_ptr + bh * (q.g + 1) + i_blk;
    // (offsets that are not what the interface asks for are brought into the head's stretch, and an entry that is no
    // block number is left out: such lists give unspecified results, but nothing outside the arrays is touched)
    const int begin = min(max(rp[0], 0), (int)cap);
    list = idx + bh * cap + begin;
    len = min(max(rp[1] - begin, 0), (int)cap - begin);
  }
  int t = -1, j = 0;
  auto advance = [&]() {
    do {
      ++t;
      j = t < len ? __builtin_amdgcn_readfirstlane(list[t]) : 0;
    } while (t < len && (unsigned)j >= (unsigned)q.g);
  };
  float4 kreg[NCH], vreg[NCH];
  auto fetch = [&]() {
    const BlockPos b = block_pos(q, j);
    const int nv = b.vh * b.vw;
    const long long first = block_first_row(q, j, b);
    const int pitch = block_row_pitch(q, b);
    const long long base = row_offset(q.in, q.H, bh, first);
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int e = tid + 256 * i, s = e / CPR, c = e % CPR;
      const int u = s / b.vw, v = s - u * b.vw;
      const long long at = base + ((long long)u * pitch + v) * q.in.sn + 4 * c;
      kreg[i] = s < nv ? *(const float4*)(K + at) : make_float4(0.f, 0.f, 0.f, 0.f);
      if (!VT) vreg[i] = s < nv ? *(const float4*)(V + at) : make_float4(0.f, 0.f, 0.f, 0.f);
      if (VT) vreg[i] = *(const float4*)(V + (bh * q.g + j) * (long long)D * 64 + 4 * e);
    }
  };
  advance();
  if (t < len) fetch();
  while (t < len) {
    const int nv = block_valid(q, j);
    __syncthreads();                                         // everyone has left the previous tile
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int e = tid + 256 * i;
      *(float4*)&ks[(e / CPR) * LD + 4 * (e % CPR)] = kreg[i];
      if (!VT) *(float4*)&vs[(e / CPR) * LD + 4 * (e % CPR)] = vreg[i];
      if (VT) {
        const int c = e >> 4, s = 4 * (e & 15);
        vs[s * LD + c] = vreg[i].x;
        vs[(s + 1) * LD + c] = vreg[i].y;
        vs[(s + 2) * LD + c] = vreg[i].z;
        vs[(s + 3) * LD + c] = vreg[i].w;
      }
    }
    __syncthreads();
    advance();
    if (t < len) fetch();
    if (!live || 32 * kh >= nv) continue;                    // nothing but pad queries, or pad keys
    f32x16 s;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
    const float* krow = ks + (32 * kh + r32) * LD + 4 * hh;
#pragma unroll
    for (int u = 0; u < D / 8; ++u) {
      const float4 a = *(const float4*)(krow + 8 * u);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, qv[u].x, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, qv[u].y, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, qv[u].z, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, qv[u].w, s, 0, 0, 0);
    }
    if (nv < 32 * kh + 32) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (32 * kh + 8 * (i >> 2) + 4 * hh + (i & 3) >= nv) s[i] = -INFINITY;   // pad keys are never attended
    }
    float mx = s[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
    mx = across_halves_max(mx);                              // finite: the half's first slot is valid
    if (__any(mx > m)) {
      const float m_new = fmaxf(m, mx);
      const float alpha = exp2f((m - m_new) * scale_log2);
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[dt][i] *= alpha;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      s[i] = exp2f((s[i] - m) * scale_log2);
      l += s[i];
    }
    const float* vrow = vs + (32 * kh + 4 * hh) * LD + NDT * r32;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float* at = vrow + (8 * (i >> 2) + (i & 3)) * LD;
      float a[NDT];
      if (NDT == 4) *(float4*)a = *(const float4*)at;
      else *(float2*)a = *(const float2*)at;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[dt], s[i], o[dt], 0, 0, 0);
    }
  }
  l = across_halves_sum(l);

  // the upper key half hands over what it has; the lower one puts the two together
  __syncthreads();
  float* part = (qh ? vs : ks) + lane * NDT;                 // [16][64][NDT] floats per query half
  float* part_ml = (qh ? vs : ks) + 16 * 64 * NDT + lane * 2;   // (64 * LD floats hold both)
  if (kh == 1) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) part[i * 64 * NDT + dt] = o[dt][i];
    part_ml[0] = m;
    part_ml[1] = l;
  }
  __syncthreads();
  if (kh == 1 || !live) return;
  const float m2 = part_ml[0], l2 = part_ml[1];
  const float m_all = fmaxf(m, m2);
  const float a1 = l > 0.f ? exp2f((m - m_all) * scale_log2) : 0.f, a2 = l2 > 0.f ? exp2f((m2 - m_all) * scale_log2) : 0.f;
  const float l_all = l * a1 + l2 * a2;
  const float inv = l_all > 0.f ? 1.0f / l_all : 0.f;        // an empty list: zero rows
  if (!has_row) return;
  float* orow = O + row_offset(q.out, q.H, bh, my_row);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    float a[NDT];
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) a[dt] = (o[dt][i] * a1 + part[i * 64 * NDT + dt] * a2) * inv;
    float* at = orow + NDT * (8 * (i >> 2) + 4 * hh + (i & 3));
    if (NDT == 4) *(float4*)at = *(const float4*)a;
    else *(float2*)at = *(const float2*)a;
  }
  if (lse && hh == 0)
    lse[qb * 64 + my_slot] = l_all > 0.f ? m_all * (float)(1.0 / sqrt((double)D)) + logf(l_all) : -INFINITY;
}

}  // namespace

// q.in / q.out / q.reordered say where the rows of Q, K (and V, unless it is block-transposed) and O are.
hipError_t launch_attn_f32(const Geo& q, const float* Q, const float* K, const float* V, bool v_transposed,
                           const int32_t* idx, const int32_t* row_ptr, long long cap, float* O, float* lse, hipStream_t s) {
  const long long total = (long long)q.B * q.H * q.g;
  const dim3 grid((unsigned)(8 * ((total + 7) / 8)));
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, q, Q, K, V, idx, row_ptr, cap, O, lse);
  };
  if (q.d == 64 && v_transposed) go(attn_f32_kernel<64, true>);
  else if (q.d == 64) go(attn_f32_kernel<64, false>);
  else if (v_transposed) go(attn_f32_kernel<128, true>);
  else go(attn_f32_kernel<128, false>);
  return hipGetLastError();
}

}  // namespace da
