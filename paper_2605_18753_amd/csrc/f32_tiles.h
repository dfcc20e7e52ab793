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
// Whether a lane of the wave holds a NaN or an infinity among these rows.
template <int D, int SUB> __device__ __forceinline__ bool any_nonfinite(const f32x4 (&rows)[SUB][4][D / 64]) {
  float z = 0.f;
#pragma unroll
  for (int st = 0; st < SUB; st++)
#pragma unroll
    for (int t = 0; t < 4; t++)
#pragma unroll
      for (int nv = 0; nv < D / 64; nv++)
#pragma unroll
        for (int e = 0; e < 4; e++) z = fmaf(rows[st][t][nv][e], 0.f, z);   // 0, or NaN
  return __any(z != z);
}
// Second kind, contraction over SUB x 16 keys that the tokens of the tile do not all attend: lane (n, hq)
// attends its row 16 st + t iff it is <= lim (lim already less 4 hq), w is 0 elsewhere.  0 times a NaN or an
// infinity is NaN, so where the rows hold one the tokens of the tile are summed one after the
// other over the keys that the token attends.  (One FMA per loaded value finds out: 1 in 50 of the time of the
// MFMAs that follow; tiles whose keys are all attended skip it.)
template <int D, int SUB> __device__ __forceinline__ void mma_outer_keys(const f32x4 (&rows)[SUB][4][D / 64], const f32x4 (&w)[SUB], int lim,
                                                                       int ntok, int g_q, int lane, f32x4 (&acc)[D / 16]) {
  if (__any(lim < 16 * SUB - 13) && any_nonfinite<D, SUB>(rows)) {
    for (int tok = 0; tok < ntok; tok++) {
      const int lt = __shfl(lim, (lane & 48) + tok * g_q);
      const bool mine = min((lane & 15) / g_q, ntok - 1) == tok;
#pragma unroll
      for (int nv = 0; nv < D / 64; nv++)
#pragma unroll
        for (int e = 0; e < 4; e++) {         // one result register group at a time: no second set of accumulators
          f32x4 sum = acc[4 * nv + e];
#pragma unroll
          for (int st = 0; st < SUB; st++)
#pragma unroll
            for (int t = 0; t < 4; t++)
              sum = __builtin_amdgcn_mfma_f32_16x16x4f32(16 * st + t <= lt ? rows[st][t][nv][e] : 0.f, w[st][t], sum, 0, 0, 0);
#pragma unroll
          for (int v = 0; v < 4; v++) acc[4 * nv + e][v] = mine ? sum[v] : acc[4 * nv + e][v];
        }
    }
    return;
  }
#pragma unroll
  for (int st = 0; st < SUB; st++)
#pragma unroll
    for (int t = 0; t < 4; t++) mma_outer<D>(rows[st][t], w[st][t], acc);
}
// The same with the roles exchanged: contraction over the 16 (token, head) rows of a tile, lane n is a key,
// `dead` says per lane and token of the tile (a bit each) whether the key is not attended by it.
template <int D> __device__ __forceinline__ void mma_outer_rows(const f32x4 (&rows)[1][4][D / 64], const f32x4& w, uint32_t dead, int g_q, int lane,
                                                                f32x4 (&acc)[D / 16]) {
  if (__any(dead != 0u) && any_nonfinite<D, 1>(rows)) {
    for (int tok = 0; tok < 16 / g_q; tok++) {
      const bool mine = !((dead >> tok) & 1u);
#pragma unroll
      for (int nv = 0; nv < D / 64; nv++)
#pragma unroll
        for (int e = 0; e < 4; e++) {
          f32x4 sum = acc[4 * nv + e];
#pragma unroll
          for (int t = 0; t < 4; t++)
            sum = __builtin_amdgcn_mfma_f32_16x16x4f32((4 * (lane >> 4) + t) / g_q == tok ? rows[0][t][nv][e] : 0.f, w[t], sum, 0, 0, 0);
#pragma unroll
          for (int v = 0; v < 4; v++) acc[4 * nv + e][v] = mine ? sum[v] : acc[4 * nv + e][v];
        }
    }
    return;
  }
#pragma unroll
  for (int t = 0; t < 4; t++) mma_outer<D>(rows[0][t], w[t], acc);
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

}  // namespace dash
