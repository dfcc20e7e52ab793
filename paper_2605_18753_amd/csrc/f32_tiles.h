// Building blocks of the kernels that multiply in fp32 on the matrix cores
// (v_mfma_f32_16x16x4_f32: fp32 products, fp32 sums; 256 flop per clock and CU): the fp32
// attention (attn_f32.hip) and the routing backward (bwd_route.hip).
//
// Tiles.  A 16-row tile holds the g_q heads of 16 / g_q consecutive tokens of one kv-head; keys
// go by 16 as well.  Both kinds of product read their operands straight from global memory (L2)
// with 16-byte loads and need no shuffle in between:
//   first kind, contraction over d (S = K Q^T, dP = V dO^T): lane (m = lane % 16, kq = lane / 16)
//     loads d = 16 s + 4 kq .. + 3 of its row m, for both operands; element e of load s is one
//     MFMA.  The result, lane (n, hq), is column n (of the B operand) at A rows 4 hq .. + 3.
//   second kind, contraction over the A rows of the first (O^T = V^T P^T, dQ^T = K^T dZ^T, dV^T =
//     dO^T P, dK^T = Q^T dZ): step t contracts the rows 4 kq + t, so lane (n, kq) supplies its own
//     accumulator register t; the other operand's lane (m, kq) loads d = 64 nv + 4 m .. + 3 of row
//     4 kq + t, element e being the d-tile {64 nv + 4 m + e}.  Result: d = 64 nv + 16 hq + 4 v + e.
#pragma once
#include "common.h"

namespace dash {

template <int D> struct F32Cfg {
  static constexpr int NS = D / 16;     // 16-byte loads of a row, first kind
  static constexpr int NV = D / 64;     // 16-byte loads of a row, second kind
  static constexpr int LD = D + 4;      // LDS row of a result tile (floats)
};

template <int D> __device__ __forceinline__ void load_row(const float* row, int kq, f32x4 (&v)[D / 16]) {
#pragma unroll
  for (int s = 0; s < D / 16; s++) v[s] = *reinterpret_cast<const f32x4*>(row + 16 * s + 4 * kq);
}
// first kind: 16 A rows x 16 B rows.  Four partial sums, added pairwise: closer to the exact sum
// than one chain of d products (rms error of a 128-term dot of N(0,1) terms 0.6e-6 against 1.15e-6).
template <int D> __device__ __forceinline__ f32x4 mma_dot(const f32x4 (&a)[D / 16], const f32x4 (&b)[D / 16]) {
  f32x4 acc[4];
#pragma unroll
  for (int i = 0; i < 4; i++) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < D / 16; s++)
#pragma unroll
    for (int e = 0; e < 4; e++) acc[s & 3] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s][e], b[s][e], acc[s & 3], 0, 0, 0);
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}
// second kind, one step t: acc[4 nv + e] += (row's d 64 nv + 4 m + e) * w
template <int D> __device__ __forceinline__ void mma_outer(const f32x4 (&row)[D / 64], float w, f32x4 (&acc)[D / 16]) {
#pragma unroll
  for (int nv = 0; nv < D / 64; nv++)
#pragma unroll
    for (int e = 0; e < 4; e++)
      acc[4 * nv + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(row[nv][e], w, acc[4 * nv + e], 0, 0, 0);
}
template <int D> __device__ __forceinline__ void load_row2(const float* row, int m, f32x4 (&v)[D / 64]) {
#pragma unroll
  for (int nv = 0; nv < D / 64; nv++) v[nv] = *reinterpret_cast<const f32x4*>(row + 64 * nv + 4 * m);
}
// a second-kind result into LDS row n of a [16][LD] tile
template <int D> __device__ __forceinline__ void put_tile(float* tile, int n, int hq, const f32x4 (&acc)[D / 16], float w) {
#pragma unroll
  for (int nv = 0; nv < D / 64; nv++)
#pragma unroll
    for (int v = 0; v < 4; v++) {
      const f32x4 x = {acc[4 * nv][v] * w, acc[4 * nv + 1][v] * w, acc[4 * nv + 2][v] * w, acc[4 * nv + 3][v] * w};
      *reinterpret_cast<f32x4*>(tile + n * F32Cfg<D>::LD + 64 * nv + 16 * hq + 4 * v) = x;
    }
}
__device__ __forceinline__ float quad_rows_max(float x) {   // over the four lanes of a column n
  x = fmaxf(x, __shfl_xor(x, 16));
  return fmaxf(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ float quad_rows_sum(float x) {
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}

}  // namespace dash
