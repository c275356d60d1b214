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

// One workgroup per (block, batch*head).  cpr = 16-byte chunks per row.
// FWD: Y[slot] = X[pi[slot]] or zeros;  !FWD: X-order output, Y[token] = Xp[slot].
// The reordered side is contiguous [B,H,n_pad,d]; the other side is the caller's tensor (q.in for
// the source of FWD, q.out for the destination of !FWD).
template <bool FWD>
__global__ __launch_bounds__(256) void permute_rows_kernel(Geo q, const chunk16* __restrict__ X, chunk16* __restrict__ Y,
                                                            int cpr) {
  int i = blockIdx.x;
  long long bh = blockIdx.y;
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

template <typename E, bool OPERAND>
__global__ __launch_bounds__(256) void permute_vt_kernel(Geo q, const E* __restrict__ X, E* __restrict__ Y) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  vt_block<E, OPERAND>(q, X, Y, (int)blockIdx.x, blockIdx.y, smem);
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
