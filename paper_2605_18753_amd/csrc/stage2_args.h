// Kernel arguments shared by the bf16 Stage-2 kernels (prefill / dense in
// stage2.hip, split-KV decode in stage2_decode.hip).
#pragma once
#include "common.h"
#include "dash_internal.h"

namespace dash {

// Estimated costs of a tile of 128 rows: of its chunks in s2_attend_kernel, of its items in s2_gather_kernel
struct S2Costs { float attend, gather; };
constexpr int kCostTiles = 64;

struct S2Args {
  const uint16_t* q; const uint16_t* k; const uint16_t* v; uint16_t* o;
  const uint32_t* mask; const float* bias;
  int h_q, h_kv, g_q, n_q, n_kv, block, t_all, words, pos0, causal, n_tiles, hb;
  int64_t qs_b, qs_h, qs_t, ks_b, ks_h, ks_t, vs_b, vs_h, vs_t, os_b, os_h, os_t;
  float c1;      // scale * log2(e)
  float* part;   // decode partials
  // prefill: parts of a workgroup's chunk list (1: not cut), their records and how many each tile has
  int max_parts; float* part_o; float* part_ml; int32_t* part_cnt;
  S2Costs* costs;   // prefill: both kernels' estimated costs of kCostTiles tiles, and the counters behind them; null: s2_attend_kernel
  const int32_t* seq_lens;   // decode: per-sequence cache lengths (device, [batch]) or null
};

constexpr float kLazy = 8.f;   // lazy-rescale slack, in base-2 logit units

inline void fill_s2_args(S2Args& a, const dash_params& p, const Layout& L, const void* q, const void* k,
                         const void* v, void* o, const uint32_t* mask, const float* bias) {
  a.q = (const uint16_t*)q; a.k = (const uint16_t*)k; a.v = (const uint16_t*)v; a.o = (uint16_t*)o;
  a.mask = mask; a.bias = bias; a.part = nullptr; a.max_parts = 1; a.part_o = a.part_ml = nullptr; a.part_cnt = nullptr; a.costs = nullptr; a.seq_lens = L.seq_lens;
  a.h_q = p.h_q; a.h_kv = p.h_kv; a.g_q = L.g_q; a.n_q = p.n_q; a.n_kv = p.n_kv;
  a.block = p.block_size; a.t_all = L.t_all; a.words = L.words; a.pos0 = L.pos0;
  a.causal = p.causal;
  a.hb = p.h_kv * p.batch;
  a.n_tiles = 1;
  a.qs_b = p.q_stride[0]; a.qs_h = p.q_stride[1]; a.qs_t = p.q_stride[2];
  a.ks_b = p.k_stride[0]; a.ks_h = p.k_stride[1]; a.ks_t = p.k_stride[2];
  a.vs_b = p.v_stride[0]; a.vs_h = p.v_stride[1]; a.vs_t = p.v_stride[2];
  a.os_b = p.o_stride[0]; a.os_h = p.o_stride[1]; a.os_t = p.o_stride[2];
  a.c1 = L.scale * kLog2e;
}

// the kernel that gathers rows (stage2_gather.hip)
bool s2_may_gather(const S2Args& a, int d);
hipError_t launch_s2_costs(const S2Args& a, int d, hipStream_t st);
hipError_t launch_s2_gather(const S2Args& a, int d, hipStream_t st);

// Whether a launch's tiles are left to s2_gather_kernel; lane i brings the costs of tile i of the kCostTiles.
__device__ __forceinline__ bool s2_gathered(S2Costs c) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) { c.attend += __shfl_xor(c.attend, o); c.gather += __shfl_xor(c.gather, o); }
  return __builtin_amdgcn_readfirstlane(c.gather < c.attend);
}

}  // namespace dash
