// Device-side helpers shared by the gfx950 kernels of the DashAttention library:
// bf16 <-> fp32 bit conversions, wave64 cross-lane reductions (DPP + bpermute),
// MFMA operand vector types.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dash {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// fp32 -> bf16 bits, round to nearest even (inputs are finite here; NaN kept NaN).
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return f32_to_bf16_bits(lo) | (f32_to_bf16_bits(hi) << 16);
}

template <typename T> struct elem;   // element loads that widen to fp32
template <> struct elem<float> {
  static constexpr int kVec = 4;     // elements per 16 bytes
  __device__ static __forceinline__ float ld(const float* p) { return *p; }
  __device__ static __forceinline__ void st(float* p, float v) { *p = v; }
};
template <> struct elem<uint16_t> {
  static constexpr int kVec = 8;
  __device__ static __forceinline__ float ld(const uint16_t* p) { return bf16_bits_to_f32(*p); }
  __device__ static __forceinline__ void st(uint16_t* p, float v) { *p = (uint16_t)f32_to_bf16_bits(v); }
};

// ---- DPP moves (wave64, rows of 16 lanes) ---------------------------------
template <int CTRL> __device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}
struct OpAdd { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };
struct OpMax { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };
// combine over the 16 lanes of a DPP row; every lane of the row gets the result
template <typename Op> __device__ __forceinline__ float row16_reduce(float v, Op op) {
  v = op(v, dpp_f<0xB1>(v));   // quad_perm [1,0,3,2]
  v = op(v, dpp_f<0x4E>(v));   // quad_perm [2,3,0,1]
  v = op(v, dpp_f<0x141>(v));  // row_half_mirror
  v = op(v, dpp_f<0x140>(v));  // row_mirror
  return v;
}
// Whole-wave combine: DPP inside each 16-lane row, then the four row results are
// read as scalars (no LDS round trip).  The result is wave-uniform by
// construction, so every decision derived from it is identical in all lanes.
template <typename Op> __device__ __forceinline__ float wave_reduce(float v, Op op) {
  v = row16_reduce(v, op);
  const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
  const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
  const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
  const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
  return op(op(r0, r1), op(r2, r3));
}
__device__ __forceinline__ float wave_sum(float v) {
  // materialise v first: a multiply contracted into the first DPP add would make
  // lane 0 of each row see a differently rounded partial sum than its partner
  asm volatile("" : "+v"(v));
  return wave_reduce(v, OpAdd());
}
__device__ __forceinline__ float wave_max(float v) { return wave_reduce(v, OpMax()); }
__device__ __forceinline__ float row16_sum(float v) { return row16_reduce(v, OpAdd()); }

// over the four lanes n, n + 16, n + 32, n + 48
__device__ __forceinline__ float quad_rows_max(float v) {
  const uint32_t u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const uint32_t w = __float_as_uint(fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1])));
  const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float quad_rows_sum(float v) {
  const uint32_t u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const uint32_t w = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
// inclusive sum over the lanes up to one's own in six DPP additions: the same through the LDS crossbar stands
// in front of the first tile of every workgroup of s2_attend_kernel (757 tokens, 32 / 8 heads of 64: 29.9 -> 28.6 us for the whole call)
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr 1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast 15: rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast 31: rows 2 and 3
  return v;
}

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63u; }

// One wave: ORs the mask rows of consecutive tokens (n = tokens * words consecutive words) into
// own[words] and own into all[words], both in LDS and zeroed by an earlier barrier.  Eight loads are in
// flight at a time: one token after the other, each load waited for, took 32 round trips to memory at 32
// tokens per wave, before the first tile of a workgroup could be copied.
__device__ __forceinline__ void or_mask_rows(const uint32_t* rows, int n, int words, uint32_t* own, uint32_t* all, int lane) {
  for (int i0 = lane; i0 - lane < n; i0 += 8 * 64) {
    uint32_t w[8];
#pragma unroll
    for (int k = 0; k < 8; k++) w[k] = i0 + 64 * k < n ? rows[i0 + 64 * k] : 0u;
#pragma unroll
    for (int k = 0; k < 8; k++)
      if (w[k]) atomicOr(&own[(i0 + 64 * k) % words], w[k]);
  }
  asm volatile("" ::: "memory");              // a wave's LDS operations complete in order
  for (int wi = lane; wi < words; wi += 64) {
    const uint32_t m = own[wi];
    if (m) atomicOr(&all[wi], m);
  }
}

// A workgroup's list of 64-key tiles from the chunk bitmaps of its rows, all[64] and waves[4][64] (in LDS, complete).  Entry: tile
// number (< 4096), bits 12 + w: wave w takes part.  Returns the number of chunks; a chunk has 1 << sub_log tiles.
template <int THREADS> __device__ __forceinline__ int list_tiles(const uint32_t* all, const uint32_t* waves, uint16_t* list, int sub_log, int tid) {
  constexpr int LPW = THREADS / 64, BPL = 32 / LPW;          // lanes per mask word, bits per lane
  const int own = __popc(all[tid & 63]);
  const int incl = wave_scan(own);
  const int wi = tid / LPW, b0 = (tid % LPW) * BPL;
  const uint32_t m = all[wi];
  int at = __shfl(incl - own, wi) + __popc(m & ((1u << b0) - 1u));
  const uint32_t w0 = waves[wi] >> b0, w1 = waves[64 + wi] >> b0, w2 = waves[128 + wi] >> b0, w3 = waves[192 + wi] >> b0;
#pragma unroll
  for (int j = 0; j < BPL; j++)
    if ((m >> (b0 + j)) & 1u) {
      const uint32_t on = ((w0 >> j) & 1u) | ((w1 >> j) & 1u) << 1 | ((w2 >> j) & 1u) << 2 | ((w3 >> j) & 1u) << 3;
      const uint32_t e = (uint32_t)((wi * 32 + b0 + j) << sub_log) | on << 12;
      list[at << sub_log] = (uint16_t)e;
      if (sub_log) list[at * 2 + 1] = (uint16_t)(e + 1);
      at++;
    }
  return __builtin_amdgcn_readlane(incl, 63);
}

}  // namespace dash
