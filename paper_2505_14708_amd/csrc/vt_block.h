// One block of the block-transposed reorder, for the kernels that do it.
#pragma once
#include <type_traits>
#include "da_internal.h"

namespace da {

typedef uint4 chunk16;  // 16 bytes

// a source chunk is read exactly once by these kernels: non-temporal, so that the stream leaves the L2 to others
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ inline chunk16 load_once(const chunk16* p) {
  const u32x4 v = __builtin_nontemporal_load((const u32x4*)p);
  return make_uint4(v.x, v.y, v.z, v.w);
}

// Block-transposed reorder: Xt[bh][i][c][s] = X[bh][pi[i*block+s]][c] (zeros in pad slots).
// A workgroup of 256 threads takes one block.  The block's rows go through LDS; ES = element bytes.
// OPERAND (bf16, block a multiple of 64, d a multiple of 32): the same transposed block, written as
// the 16-byte operands of the matrix instructions, one 64-slot sub-block after the other: unit
// ((t*nd + dt)*64 + hh*32 + r) of sub-block sb holds channel 32dt + r, slots 64sb + 16t + 8hh + 0..7.
template <typename E, bool OPERAND>
__device__ __forceinline__ void vt_block(const Geo& q, const E* __restrict__ X, E* __restrict__ Y, int i, long long bh,
                                         unsigned char* smem) {
  constexpr int PER = 16 / sizeof(E);  // elements per 16-byte chunk
  E* tile = (E*)smem;                  // [block][d + PER] (padded rows)
  const int ld = q.d + PER;
  BlockPos b = block_pos(q, i);
  int nv = b.vh * b.vw;
  int cpr = q.d / PER;
  const chunk16* Xc = (const chunk16*)(X + row_offset(q.in, q.H, bh, block_first_row(q, i, b)));   // the block's first row
  const long long sn = q.in.sn / PER, pitch = block_row_pitch(q, b);
  // A thread's four chunks of a 16 KB block are all on their way before the first is put down: 12.3 -> 11.3 us at 1344 blocks,
  // 15.2 -> 14.0 us at 2016; larger launches as before, where other workgroups fill the waits.  Blocks of no more than a chunk
  // per thread (4x4 windows, say) have nothing to ask for ahead: 7920 of them with 8 heads 103.5 -> 100 us one at a time.
  auto bring = [&](auto ahead) {
    constexpr int AHEAD = decltype(ahead)::value;
    for (int e0 = threadIdx.x; e0 < q.block * cpr; e0 += AHEAD * 256) {
      chunk16 val[AHEAD];
#pragma unroll
      for (int j = 0; j < AHEAD; ++j) {
        const int e = e0 + 256 * j, s = e / cpr, c = e - s * cpr;
        val[j] = make_uint4(0, 0, 0, 0);
        if (s < nv) {                                  // (nv <= block: such an e is below block * cpr as well)
          const int u = s / b.vw, v = s - u * b.vw;
          val[j] = load_once(&Xc[((long long)u * pitch + v) * sn + c]);
        }
      }
#pragma unroll
      for (int j = 0; j < AHEAD; ++j) {
        const int e = e0 + 256 * j, s = e / cpr, c = e - s * cpr;
        if (s < q.block) *(chunk16*)(tile + s * ld + c * PER) = val[j];
      }
    }
  };
  if (q.block * cpr > 256) bring(std::integral_constant<int, 4>());
  else bring(std::integral_constant<int, 1>());
  __syncthreads();
  E* out = Y + (bh * q.g + i) * (long long)q.d * q.block;
  if (OPERAND) {
    const int nd = q.d >> 5, per_half = q.d * 64 / PER;   // 16-byte units per 64-slot sub-block
    for (int e = threadIdx.x; e < q.d * q.block / PER; e += blockDim.x) {
      const int sb = e / per_half, eh = e - sb * per_half;
      const int r = eh & 31, hh = (eh >> 5) & 1, grp = eh >> 6;
      const int t = grp / nd, dt = grp - t * nd;
      const int c = 32 * dt + r, s0 = 64 * sb + 16 * t + 8 * hh;
      E tmp[PER];
#pragma unroll
      for (int j = 0; j < PER; ++j) tmp[j] = tile[(s0 + j) * ld + c];
      *(chunk16*)(out + (long long)e * PER) = *(chunk16*)tmp;
    }
    return;
  }
  int spr = q.block / PER;  // 16-byte chunks per output row (a row holds `block` slots of one channel)
  for (int e = threadIdx.x; e < q.d * spr; e += blockDim.x) {
    int c = e / spr, s8 = e - c * spr;
    E tmp[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) tmp[j] = tile[(s8 * PER + j) * ld + c];
    *(chunk16*)(out + (long long)c * q.block + s8 * PER) = *(chunk16*)tmp;
  }
}

// LDS that takes
inline size_t vt_block_lds(const Geo& q) {
  const size_t es = q.dtype == DA_BF16 ? 2 : 4;
  return (size_t)q.block * (q.d + 16 / es) * es;
}

}  // namespace da
