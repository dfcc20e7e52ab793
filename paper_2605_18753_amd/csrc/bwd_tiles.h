// LDS tiles and operand reads shared by the bf16 backward kernels (backward.hip, bwd_kv.hip).
#pragma once
#include "common.h"
#include "lds_copy.h"

namespace dash {

template <int D> struct BCfg {
  static constexpr int NCH = D / 8;
  static constexpr int ROW_BYTES = D * 2;
  static constexpr int TILE_BYTES = 64 * ROW_BYTES;
  static constexpr int COPIES = TILE_BYTES / 16 / 256;
  static constexpr int ROWS_PER_COPY = 256 / NCH;
  static constexpr int NDT = D / 32;
  static constexpr int NS = D / 8;
};

// Chunk permutation of a 64-row tile (position of logical 16-byte chunk c of row
// `row` is c ^ swz(row)), chosen so that both kinds of operand reads are free of
// bank conflicts: the A-operand read has 16 lanes on 16 consecutive rows at one
// logical chunk (they must land in 16 different slots of a 256-byte bank window),
// the transposing read has 16 lanes on 4 consecutive rows x 2 consecutive chunks
// (rows r..r+3 must land in different 64-byte groups).
template <int D> __device__ __forceinline__ int swz(int row) {
  return D == 128 ? (((row & 3) << 2) | ((row >> 2) & 3)) : ((((row >> 1) & 1) << 2) | ((row >> 2) & 3));
}
// byte offset of element (row, d0) of a tile, d0 a multiple of 4
template <int D> __device__ __forceinline__ uint32_t tile_off(int row, int d0) {
  return (uint32_t)(row * BCfg<D>::ROW_BYTES + (((d0 >> 3) ^ swz<D>(row)) << 4) + ((d0 & 7) << 1));
}

// Operand addresses.  Because the chunk permutation is an XOR, the offsets of the
// d slices of one row differ from the first one by an XOR with a constant, so a
// lane keeps one base offset per kind of read instead of one register per slice.
// A operand slice `i` (d slice ks = i / 2, 32-row half i % 2) of a row-major tile;
// base = tile_off(row, 8 h): the slice starts at d = 16 ks + 8 h, chunk 2 ks + h
template <int D> __device__ __forceinline__ bf16x8 read_a(const char* tile, uint32_t base, int i) {
  return *reinterpret_cast<const bf16x8*>(tile + (base ^ (uint32_t)((i >> 1) << 5)) + (i & 1) * 32 * BCfg<D>::ROW_BYTES);
}
// transposed A operand: contraction step g (16 tile rows), d-tile t; lo / hi address the
// two 8-row halves of step 0 at d-tile 0 (d-tile t starts 4 t chunks further)
template <int D> __device__ __forceinline__ bf16x8 read_t(const char* tile, uint32_t lo, uint32_t hi, int g, int t) {
  return lds_read_tr_pair(tile + (lo ^ (uint32_t)(t << 6)) + (16 * g) * BCfg<D>::ROW_BYTES,
                          tile + (hi ^ (uint32_t)(t << 6)) + (16 * g) * BCfg<D>::ROW_BYTES);
}

__device__ __forceinline__ f32x16 zero16() {
  const f32x16 z = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  return z;
}

}  // namespace dash
