// Reordering by pi (Algorithm 1) and restoring by pi^-1 (Algorithm 2) as pure data movement.
// HBM-bound: every element is read once and written once in 16-byte pieces; the index
// arithmetic is done on the fly, no index array is read.
#include "da_internal.h"
#include "vt_block.h"

namespace da {

// perm / inv / valid arrays for callers that want them.
__global__ void build_perm_kernel(Geo q, int32_t* perm, int32_t* inv, int32_t* valid) {
  long long slot = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (slot >= q.n_pad) return;
  int i = (int)(slot / q.block);
  int s = (int)(slot - (long long)i * q.block);
  BlockPos b = block_pos(q, i);
  int nv = b.vh * b.vw;
  int tok = -1;
  if (s < nv) {
    int u = s / b.vw, v = s - u * b.vw;
    tok = (b.f * q.fh + b.y0 + u) * q.fw + b.x0 + v;
    if (inv) inv[tok] = (int32_t)slot;
  }
  if (perm) perm[slot] = tok;
  if (valid && s == 0) valid[i] = nv;
}

// A workgroup of 256 threads takes one block.  cpr = 16-byte chunks per row.
// FWD: Y[slot] = X[pi[slot]] or zeros;  !FWD: X-order output, Y[token] = Xp[slot].
// The reordered side is contiguous [B,H,n_pad,d]; the other side is the caller's tensor (q.in for
// the source of FWD, q.out for the destination of !FWD).
template <bool FWD>
__device__ __forceinline__ void rows_block(const Geo& q, const chunk16* __restrict__ X, chunk16* __restrict__ Y, int cpr, int i,
                                           long long bh) {
  BlockPos b = block_pos(q, i);
  int nv = b.vh * b.vw;
  const int per = q.d / cpr;                           // elements per chunk
  const Rows& far = FWD ? q.in : q.out;
  const long long far0 = row_offset(far, q.H, bh, block_first_row(q, i, b)) / per;   // chunk of the block's first row
  const long long far_sn = far.sn / per, pitch = block_row_pitch(q, b);
  const long long near0 = (bh * q.n_pad + (long long)i * q.block) * cpr;
  int total = (FWD ? q.block : nv) * cpr;
  for (int e = threadIdx.x; e < total; e += blockDim.x) {
    int s = e / cpr, c = e - s * cpr;
    if (FWD) {
      chunk16 val = make_uint4(0, 0, 0, 0);
      if (s < nv) {
        int u = s / b.vw, v = s - u * b.vw;
        val = load_once(&X[far0 + ((long long)u * pitch + v) * far_sn + c]);
      }
      Y[near0 + (long long)s * cpr + c] = val;
    } else {
      int u = s / b.vw, v = s - u * b.vw;
      Y[far0 + ((long long)u * pitch + v) * far_sn + c] = load_once(&X[near0 + (long long)s * cpr + c]);
    }
  }
}

template <bool FWD>
__global__ __launch_bounds__(256) void permute_rows_kernel(Geo q, const chunk16* __restrict__ X, chunk16* __restrict__ Y,
                                                            int cpr) {
  rows_block<FWD>(q, X, Y, cpr, (int)blockIdx.x, blockIdx.y);
}

template <typename E, bool OPERAND>
__global__ __launch_bounds__(256) void permute_vt_kernel(Geo q, const E* __restrict__ X, E* __restrict__ Y) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  vt_block<E, OPERAND>(q, X, Y, (int)blockIdx.x, blockIdx.y, smem);
}

// All that stands before the attention where every block is kept (bf16): the reordering of V, that of K (Kp NULL: it stays where
// it is) and the lists 0 .. g-1, in one launch, a workgroup for each block and each list.
// da_forward and da_forward_global, us, three launches (two with K in place) -> one: 2 heads of a 30x52 frame 39.3 -> 34.4, 24 of
// them 73.1 -> 67.3, in block order 65.6 -> 63.5, 8 heads of two 45x80 frames 240 -> 234, 24 of nine 30x52 frames 2571 -> 2557.
__global__ __launch_bounds__(256) void prepare_dense_kernel(Geo q, const chunk16* __restrict__ K, const uint16_t* __restrict__ V,
                                                            chunk16* __restrict__ Kp, uint16_t* __restrict__ Vt,
                                                            int32_t* __restrict__ idx, int32_t* __restrict__ row_ptr,
                                                            long long head_stride, int cpr) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const unsigned what = blockIdx.y, b = blockIdx.x;
  const unsigned bh = b / (unsigned)q.g;
  const int i = (int)(b - bh * (unsigned)q.g);
  if (what == 0) {
    vt_block<uint16_t, true>(q, V, Vt, i, bh, smem);
  } else if (what == 1 && Kp) {
    rows_block<true>(q, K, Kp, cpr, i, bh);
  } else {
    for (int j = threadIdx.x; j < q.g; j += 256) idx[bh * head_stride + (long long)i * q.g + j] = j;
    if (row_ptr && threadIdx.x == 0) {
      row_ptr[bh * (long long)(q.g + 1) + i] = i * q.g;
      if (i == q.g - 1) row_ptr[bh * (long long)(q.g + 1) + q.g] = q.g * q.g;
    }
  }
}

hipError_t launch_prepare_dense(const Geo& q, const void* K, const void* V, void* Kp, void* Vt, int32_t* idx, int32_t* row_ptr,
                                long long head_stride, hipStream_t s) {
  // (a launch has fewer than 2^32 threads along an axis: along x alone six million blocks would be too many)
  const unsigned blocks = (unsigned)((long long)q.B * q.H * q.g);
  hipLaunchKernelGGL(prepare_dense_kernel, dim3(blocks, Kp ? 3 : 2), dim3(256), vt_block_lds(q), s, q, (const chunk16*)K,
                     (const uint16_t*)V, (chunk16*)Kp, (uint16_t*)Vt, idx, row_ptr, head_stride, q.d / 8);
  return hipGetLastError();
}

hipError_t launch_build_perm(const Geo& q, int32_t* perm, int32_t* inv, int32_t* valid, hipStream_t s) {
  unsigned blocks = (unsigned)((q.n_pad + 255) / 256);
  hipLaunchKernelGGL(build_perm_kernel, dim3(blocks), dim3(256), 0, s, q, perm, inv, valid);
  return hipGetLastError();
}

hipError_t launch_permute(const Geo& q, const void* X, void* Y, int mode, hipStream_t s) {
  size_t es = q.dtype == DA_BF16 ? 2 : 4;
  int cpr = (int)(q.d * es / 16);
  dim3 grid((unsigned)q.g, (unsigned)(q.B * q.H));
  if (mode == DA_REORDER_ROWS) {
    hipLaunchKernelGGL(permute_rows_kernel<true>, grid, dim3(256), 0, s, q, (const chunk16*)X, (chunk16*)Y, cpr);
  } else if (mode == DA_RESTORE) {
    hipLaunchKernelGGL(permute_rows_kernel<false>, grid, dim3(256), 0, s, q, (const chunk16*)X, (chunk16*)Y, cpr);
  } else {
    const size_t lds = vt_block_lds(q);
    if (lds > 64 * 1024) return hipErrorInvalidValue;
    if (mode == DA_REORDER_VOP)
      hipLaunchKernelGGL((permute_vt_kernel<uint16_t, true>), grid, dim3(256), lds, s, q, (const uint16_t*)X, (uint16_t*)Y);
    else if (es == 2)
      hipLaunchKernelGGL((permute_vt_kernel<uint16_t, false>), grid, dim3(256), lds, s, q, (const uint16_t*)X, (uint16_t*)Y);
    else
      hipLaunchKernelGGL((permute_vt_kernel<uint32_t, false>), grid, dim3(256), lds, s, q, (const uint32_t*)X, (uint32_t*)Y);
  }
  return hipGetLastError();
}

}  // namespace da
