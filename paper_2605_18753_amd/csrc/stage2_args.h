// Kernel arguments shared by the bf16 Stage-2 kernels (prefill / dense in
// stage2.hip, split-KV decode in stage2_decode.hip).
#pragma once
#include "common.h"
#include "dash_internal.h"

namespace dash {

// What a launch that s2_attend_kernel or s2_gather_kernel may take knows of its lists.  The records lie in the library, not in the caller's
// workspace, into which such a launch writes nothing, and are dealt out in turn (kChoices of them).  Of kCostTiles tiles: the number of the
// call (high word) and what the tile is estimated to cost in s2_gather_kernel beyond s2_attend_kernel (fp32, low word), in one store.  A record
// that also serves another call in flight shows that call's number sooner or later, and never this call's again: then either kernel attends,
// the second over the first.  They leave tiles out only where the whole record is their own, and then both find the same sum.
constexpr int kCostTiles = 64;
struct S2Choice {
  uint64_t costs[kCostTiles];
  int arrived[8 * 32];        // workgroups of s2_gather_kernel that began, by die
};

struct S2Args {
  const uint16_t* q; const uint16_t* k; const uint16_t* v; uint16_t* o;
  const uint32_t* mask; const float* bias;
  int h_q, h_kv, g_q, n_q, n_kv, block, t_all, words, pos0, causal, n_tiles, hb;
  int64_t qs_b, qs_h, qs_t, ks_b, ks_h, ks_t, vs_b, vs_h, vs_t, os_b, os_h, os_t;
  float c1;      // scale * log2(e)
  float* part;   // decode partials
  // prefill: parts of a workgroup's chunk list (1: not cut), their records and how many each tile has
  int max_parts; float* part_o; float* part_ml; int32_t* part_cnt;
  S2Choice* choice; uint32_t call;   // prefill: the launch's record and the call's number in it; null: s2_attend_kernel
  const int32_t* seq_lens;   // decode: per-sequence cache lengths (device, [batch]) or null
};

constexpr float kLazy = 8.f;   // lazy-rescale slack, in base-2 logit units

inline void fill_s2_args(S2Args& a, const dash_params& p, const Layout& L, const void* q, const void* k,
                         const void* v, void* o, const uint32_t* mask, const float* bias) {
  a.q = (const uint16_t*)q; a.k = (const uint16_t*)k; a.v = (const uint16_t*)v; a.o = (uint16_t*)o;
  a.mask = mask; a.bias = bias; a.part = nullptr; a.max_parts = 1; a.part_o = a.part_ml = nullptr; a.part_cnt = nullptr; a.choice = nullptr; a.call = 0; a.seq_lens = L.seq_lens;
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
void s2_take_choice(S2Args& a);
hipError_t launch_s2_costs(const S2Args& a, int d, hipStream_t st);
hipError_t launch_s2_gather(const S2Args& a, int d, hipStream_t st);

// One wave: what the record says, s2_attend_kernel (< 0), s2_gather_kernel (> 0), or nothing to this call (0).
__device__ __forceinline__ int s2_choice(const S2Args& a, int lane) {
  const uint64_t x = __hip_atomic_load(&a.choice->costs[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const bool own = __all((uint32_t)(x >> 32) == a.call);
  const float more = wave_sum(__uint_as_float((uint32_t)x));
  return __builtin_amdgcn_readfirstlane(!own ? 0 : more < 0.f ? 1 : -1);
}

}  // namespace dash
