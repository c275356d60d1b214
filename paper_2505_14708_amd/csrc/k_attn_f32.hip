// SparseAttn for float32 storage, blocks of 64 slots, d = 64 or 128: float32 throughout, on the float32 matrix
// instructions (v_mfma_f32_16x16x4_f32: exact products, one rounding per term, like a chain of fused multiply-adds).
//
// A workgroup is half a query block, 32 queries, or a quarter where that fills the chip better (f32_share.h); its waves share
// out the keys, 16 (a quarter of a block) at a time, and keep a running maximum, a sum and an output of their own, which are put
// together at the end.  A key is then wanted by one wave only, so K and V go straight from memory to that wave's registers: no
// tile in LDS, no barrier in the loop.
// Wave: 16 keys x 32 queries per step, the query on the lane axis of both products:
//     S^T = K Q^T      lane l: query l % 16 of each 16; accumulator register r: key 4(l/16) + r
//     O^T += V^T P^T   register r of P is, as it stands, the operand of the step that adds the keys 4(l/16) + r: no
//                      exchange between lanes
// Channels are taken in whatever order makes the loads wide: a 16-byte piece of a K row serves four steps of the first
// product (channels 16u + 4(l/16) + 0..3), and row i of accumulator dt of the second is channel (d/16) i + dt.
//
// What bounds it: the matrix instructions (32 cycles each; 128 of them per step and SIMD at d = 128 against 16 KB brought in).  The
// next step's K is asked for when this step's first product is through with its registers, V when the last second
// product is: each has half a step (2048 cycles) to arrive.  Half blocks because the launch is small as a rule: 84 blocks
// x 4 heads are 1.3 whole blocks per CU, and a CU with two of them set the time.  Measured against whole blocks with
// K and V tiles in LDS, two query halves by two key halves (kernel times): 226 -> 185 us at 84 blocks x 4 heads, d = 128,
// 21 blocks kept, 17.7 -> 12.2 us at 8 blocks x 2 heads, d = 64, 4 kept; da_forward with 24 heads 862 -> 769 us (116
// TFLOP/s of the 130 that a bare loop of float32 matrix instructions reaches).  Eight waves per workgroup instead of four
// gain nothing on the small ones and lose 20 % on the large ones, where two workgroups per CU hide each other's ends.
#include <float.h>
#include <math.h>
#include "da_internal.h"
#include "f32_share.h"

namespace da {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// over the four lanes that hold the same query (l, l ^ 16, l ^ 32, l ^ 48)
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float query_max(float x) {
  u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float query_sum(float x) {
  u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// VT: V comes block-transposed (DA_REORDER_VT); otherwise K and V alike are rows that q.in says where to find.
constexpr int W = 4;                         // waves of a workgroup

// What a workgroup shares with itself: the waves' outputs, references and normalisers
template <int D>
struct Parts {
  float4 out[W][2 * (D / 16)][64];
  float2 ml[W][2][16];
};

// 16 NH queries, from slot `first_query` of query block qb on
template <int D, bool VT, int NH>
__device__ __forceinline__ void attend(const Geo& q, const float* __restrict__ Q, const float* __restrict__ K,
                                       const float* __restrict__ V, const int32_t* __restrict__ idx,
                                       const int32_t* __restrict__ row_ptr, long long cap, float* __restrict__ O,
                                       float* __restrict__ lse, long long qb, int first_query, Parts<D>& parts) {
  constexpr int NU = D / 16;                 // 16-byte pieces of a K or Q row per lane
  constexpr int NDT = D / 16;                // accumulators of the second product per 16 queries
  constexpr int NG = NH * NDT;               // 16-byte groups of a lane's output
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, kk = lane >> 4;
  const long long bh = qb / q.g;
  const int i_blk = (int)(qb - bh * q.g);
  const float scale_log2 = (float)(1.4426950408889634 / sqrt((double)D));

  // query rows (slots past the valid ones exist only where the tensors are in block order)
  const BlockPos qp = block_pos(q, i_blk);
  const int q_valid = q.reordered ? 64 : qp.vh * qp.vw;      // slots with a row of their own
  if (first_query >= q_valid) return;                         // (the whole workgroup)
  const long long q_first = block_first_row(q, i_blk, qp);
  const int q_pitch = block_row_pitch(q, qp);
  auto query_row = [&](int slot) -> long long { return q_first + (long long)(slot / qp.vw) * q_pitch + slot % qp.vw; };
  float4 qv[NH][NU];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    const int slot = first_query + 16 * h + r16;
    const float* qrow = Q + row_offset(q.in, q.H, bh, query_row(slot < q_valid ? slot : 0)) + 4 * kk;
#pragma unroll
    for (int u = 0; u < NU; ++u) qv[h][u] = *(const float4*)(qrow + 16 * u);
  }
  f32x4 o[NH][NDT];
  float m[NH], l[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) o[h][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    l[h] = 0.f;
  }

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
  // The wave's steps: a quarter of every entry; which quarter goes round, so that blocks with fewer than 64 valid slots
  // cost all waves alike.  64 entries of the list are held at a time, entry t in lane t % 64, with what a step wants to
  // know of the block worked out once for all 64 (a step has little room for divisions beside its matrix instructions).
  int t = -1, held = -64;
  int e_block = 0, e_shape = 0;                              // block number; valid slots | patch columns << 8 | 65536 / columns, rounded up << 15
  unsigned e_row_lo = 0u, e_row_hi = 0u;                     // the block's first row
  int j = 0, first_key = 0, nv = 1, vw = 1, recip = 0;       // the step: block, first slot, the block's valid slots, columns
  long long first_row = 0;
  auto advance = [&]() -> bool {
    for (;;) {
      if (++t >= len) return false;
      if (t - held >= 64) {
        held = t & ~63;
        e_block = list[min(held + lane, len - 1)];
        const BlockPos b = block_pos(q, (unsigned)e_block < (unsigned)q.g ? e_block : 0);
        const long long row = block_first_row(q, (unsigned)e_block < (unsigned)q.g ? e_block : 0, b);
        e_shape = b.vh * b.vw | b.vw << 8 | (int)((unsigned)((65536 + b.vw - 1) / b.vw) << 15);
        e_row_lo = (unsigned)row;
        e_row_hi = (unsigned)(row >> 32);
        asm volatile("" : "+v"(e_block), "+v"(e_shape));     // (the load is waited for here, not with the tile loads in flight)
      }
      const int e = __builtin_amdgcn_readlane(e_block, t & 63);
      if ((unsigned)e >= (unsigned)q.g) continue;
      const int shape = __builtin_amdgcn_readlane(e_shape, t & 63);
      const int at = 16 * ((wave + t) & 3);
      if (at >= (shape & 255)) continue;
      j = e;
      first_key = at;
      nv = shape & 255;
      vw = (shape >> 8) & 127;
      recip = (unsigned)shape >> 15;
      first_row = (long long)((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)e_row_hi, t & 63) << 32 |
                              (unsigned)__builtin_amdgcn_readlane((int)e_row_lo, t & 63));
      return true;
    }
  };
  const long long head_row = row_offset(q.in, q.H, bh, 0);
  // element offset of slot `slot` of the step's block (slot / vw by way of the reciprocal: exact below 128 for vw <= 64)
  auto key_at = [&](int slot) -> long long {
    const int s = min(slot, nv - 1);                         // (a pad slot has no row of its own)
    const int u = (s * recip) >> 16;
    return (long long)(u * ((q.reordered ? vw : q.fw) - vw) + s) * q.in.sn;
  };
  float4 kr[NU];
  f32x4 vr[4][NDT / 4];                                      // !VT: [key r][channels]; VT: dt = 4 a + b is [b][a], keys in the vector
  auto fetch_k = [&]() {
    const float* at = K + head_row + first_row * q.in.sn + key_at(first_key + r16) + 4 * kk;
#pragma unroll
    for (int u = 0; u < NU; ++u) kr[u] = *(const float4*)(at + 16 * u);
  };
  auto fetch_v = [&]() {
    if (VT) {
      const float* at = V + (bh * q.g + j) * (long long)D * 64 + (long long)NDT * r16 * 64 + first_key + 4 * kk;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) vr[dt & 3][dt >> 2] = *(const f32x4*)(at + dt * 64);
    } else {
      const float* base = V + head_row + first_row * q.in.sn + NDT * r16;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float* at = base + key_at(first_key + 4 * kk + r);
#pragma unroll
        for (int a = 0; a < NDT / 4; ++a) vr[r][a] = *(const f32x4*)(at + 4 * a);
      }
    }
  };
  bool more = advance();
  // The reference of a wave that has keys starts at the lowest finite value, not at minus infinity: all scores of its first
  // steps may be minus infinity (finite operands whose product leaves the range), and those keys weigh exp2(-inf) = 0,
  // not exp2(-inf + inf).
#pragma unroll
  for (int h = 0; h < NH; ++h) m[h] = more ? -FLT_MAX : -INFINITY;
  if (more) fetch_k();
  while (more) {
    fetch_v();
    __builtin_amdgcn_sched_barrier(0);
    const int keys = nv - first_key;                         // valid keys of this step (16 or more: all of them)
    f32x4 s[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) s[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const float a[4] = {kr[u].x, kr[u].y, kr[u].z, kr[u].w};
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int h = 0; h < NH; ++h) {
          const float b = c == 0 ? qv[h][u].x : c == 1 ? qv[h][u].y : c == 2 ? qv[h][u].z : qv[h][u].w;
          s[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c], b, s[h], 0, 0, 0);
        }
    }
    if (keys < 16) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int h = 0; h < NH; ++h)
          if (4 * kk + r >= keys) s[h][r] = -INFINITY;       // pad keys are never attended
    }
    more = advance();
    __builtin_amdgcn_sched_barrier(0);
    fetch_k();                                               // (after the last step its own once more: what is in flight is then the same on every path)
    __builtin_amdgcn_sched_barrier(0);
    float mx[NH];
    bool moves = false;
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      mx[h] = query_max(fmaxf(fmaxf(s[h][0], s[h][1]), fmaxf(s[h][2], s[h][3])));
      moves = moves || mx[h] > m[h];
    }
    if (__any(moves)) {
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        const float m_new = fmaxf(m[h], mx[h]);
        const float alpha = m[h] == m_new ? 1.f : exp2f((m[h] - m_new) * scale_log2);
        m[h] = m_new;
        l[h] *= alpha;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) o[h][dt] *= alpha;
      }
    }
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[h][r] = exp2f((s[h][r] - m[h]) * scale_log2);
        l[h] += s[h][r];
      }
    if (!VT && keys < 16) {                                  // (a probability of 0 times whatever was read there)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (4 * kk + r >= keys) {
#pragma unroll
          for (int a = 0; a < NDT / 4; ++a) vr[r][a] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
        const float a = VT ? vr[dt & 3][dt >> 2][r] : vr[r][dt >> 2][dt & 3];
#pragma unroll
        for (int h = 0; h < NH; ++h) o[h][dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, s[h][r], o[h][dt], 0, 0, 0);
      }
  }

  // every wave hands over what it has; wave w puts together its share of the output's groups
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    const float lt = query_sum(l[h]);
    if (kk == 0) parts.ml[wave][h][r16] = make_float2(m[h], lt);
    // register r of accumulator dt is channel (d/16)(4 kk + r) + dt: with f = (d/16) r + dt the lane holds channels
    // (d/4) kk + f of its query
#pragma unroll
    for (int gi = 0; gi < NDT; ++gi) {
      float x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = o[h][(4 * gi + i) % NDT][(4 * gi + i) / NDT];
      parts.out[wave][h * NDT + gi][lane] = make_float4(x[0], x[1], x[2], x[3]);
    }
  }
  __syncthreads();
  constexpr int SHARE = NG / W;
  const int h = wave / (W / NH);                             // which 16 queries the wave's groups belong to
  float a[W], m_all = -INFINITY, l_all = 0.f;
#pragma unroll
  for (int w = 0; w < W; ++w) m_all = fmaxf(m_all, parts.ml[w][h][r16].x);
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const float2 ml = parts.ml[w][h][r16];
    a[w] = ml.y > 0.f ? exp2f((ml.x - m_all) * scale_log2) : 0.f;
    l_all += ml.y * a[w];
  }
  // an empty list: zero rows; keys that all score minus infinity (or NaN): no softmax is defined, NaN
  const float inv = l_all > 0.f ? 1.0f / l_all : m_all == -INFINITY ? 0.f : NAN;
  const int slot = first_query + 16 * h + r16;
  if (slot >= q_valid) return;
  float* orow = O + row_offset(q.out, q.H, bh, query_row(slot)) + (D / 4) * kk;
#pragma unroll
  for (int i = 0; i < SHARE; ++i) {
    const int grp = wave * SHARE + i;
    float4 y = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float4 x = parts.out[w][grp][lane];
      y.x += x.x * a[w];
      y.y += x.y * a[w];
      y.z += x.z * a[w];
      y.w += x.w * a[w];
    }
    *(float4*)(orow + 4 * (grp - h * NDT)) = make_float4(y.x * inv, y.y * inv, y.z * inv, y.w * inv);
  }
  if (lse && kk == 0 && wave % (W / NH) == 0)
    lse[qb * 64 + slot] = l_all > 0.f ? m_all * (float)(1.0 / sqrt((double)D)) + logf(l_all) : -INFINITY;
}

template <int D, bool VT>
__global__ __launch_bounds__(64 * W, 2) void attn_f32_kernel(Geo q, const float* __restrict__ Q, const float* __restrict__ K,
                                                             const float* __restrict__ V, const int32_t* __restrict__ idx,
                                                             const int32_t* __restrict__ row_ptr, long long cap,
                                                             float* __restrict__ O, float* __restrict__ lse, F32Share share) {
  __shared__ Parts<D> parts;
  const F32Piece piece = f32_piece(share, blockIdx.x);
  if (piece.half >= 2LL * q.B * q.H * q.g) return;           // (the last stretch may be shorter)
  const int first_query = 32 * (int)(piece.half & 1) + 16 * piece.second;
  if (piece.queries == 32) attend<D, VT, 2>(q, Q, K, V, idx, row_ptr, cap, O, lse, piece.half >> 1, first_query, parts);
  else attend<D, VT, 1>(q, Q, K, V, idx, row_ptr, cap, O, lse, piece.half >> 1, first_query, parts);
}

}  // namespace

// q.in / q.out / q.reordered say where the rows of Q, K (and V, unless it is block-transposed) and O are.
hipError_t launch_attn_f32(const Geo& q, const float* Q, const float* K, const float* V, bool v_transposed,
                           const int32_t* idx, const int32_t* row_ptr, long long cap, float* O, float* lse, hipStream_t s) {
  // (in block order every slot is a query's; else the last patches of a row, a column or both may have too few)
  const int last_h = (q.fh - 1) % q.ph + 1, last_w = (q.fw - 1) % q.pw + 1;
  const bool even = !row_ptr && (q.reordered || (last_h * last_w > 32 && last_h * q.pw > 32 && q.ph * last_w > 32));
  const F32Share share = f32_share_out(2LL * q.B * q.H * q.g, even, q.d);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(share.grid), dim3(64 * W), 0, s, q, Q, K, V, idx, row_ptr, cap, O, lse, share);
  };
  if (q.d == 64 && v_transposed) go(attn_f32_kernel<64, true>);
  else if (q.d == 64) go(attn_f32_kernel<64, false>);
  else if (v_transposed) go(attn_f32_kernel<128, true>);
  else go(attn_f32_kernel<128, false>);
  return hipGetLastError();
}

}  // namespace da
