// Arguments of the backward kernels (backward.hip, attn_f32.hip) and the launchers of the fp32 ones.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dash {

struct BwdArgs {
  const uint16_t *q, *k, *v, *d_o;
  uint16_t *dq, *dk, *dv;
  const float* kbar; const uint32_t* mask; const float* bias; const float* tau;
  float *lse, *dsum;       // [batch, h_q, n_q]: base-2 log-sum-exp of the logits, <dO, o>
  float *biasd, *dbd;      // [batch, h_kv, n_q, t_all]: bias and its gradient by chunk id
  float* dxd;              // [batch, h_q, n_q, t_all]: entmax-score gradient by chunk id
  float* dq32;             // [batch, h_q, n_q, D]: attention part of dq
  uint32_t* colmask;       // [batch*h_kv, t_all, cwords]: bit T set iff 32-row tile T attends the chunk
  float* dkbar;            // [kb_parts][batch*h_kv, t_c, D]: partial sums of the summaries' gradient
  float* kv_part;          // [key tile][batch*h_kv][kv_max_parts][2][128][D]: partial sums of dk, dv
  int kv_steps, kv_max_parts, kb_parts;   // how the key side is cut (bwd_kv.hip)
  int64_t kb_stride;       // floats of one dkbar part
  float* dkbar_out;        // optional [batch, h_kv, t_c, D]: gradient of the summaries (then not folded into dk)
  int h_q, h_kv, g_q, n_q, n_kv, block, t_c, t_all, words, causal, window, n_tiles, hb, cwords;
  int64_t qs_b, qs_h, qs_t, ks_b, ks_h, ks_t, vs_b, vs_h, vs_t, os_b, os_h, os_t;
  float c1, scale, xscale, pexp, sigma;
};

// routing backward of both data types (bwd_route.hip)
hipError_t launch_bwd_route(const BwdArgs& a, int head_dim, bool bf16, hipStream_t st);
// key side of the bf16 backward: its cut, and its launches (bwd_kv.hip)
void bwd_kv_plan(BwdArgs& a);
hipError_t launch_bwd_kv(const BwdArgs& a, int head_dim, hipStream_t st);
// fp32 tensors: row log-sum-exp, D, bias gradient and the attention part of dq; then, after the
// routing kernel, dk, dv and the summary gradient
hipError_t launch_bwd_f32_rows(const BwdArgs& a, int head_dim, hipStream_t st);
hipError_t launch_bwd_f32_keys(const BwdArgs& a, int head_dim, hipStream_t st);

}  // namespace dash
