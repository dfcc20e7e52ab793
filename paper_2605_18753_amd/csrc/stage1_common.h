// Shared by the Stage-1 kernels (stage1.hip, stage1_regs.hip): kernel arguments, the
// entmax exponent modes and the power terms of the threshold equation (Eq. 2; Alg. 2).
#pragma once
#include "common.h"

namespace dash {

struct S1Args {
  const void* q;
  const uint16_t* ksplit;
  const float* scores;
  const float* kbar;         // fp32 summaries (the decode kernel scores against them itself)
  // decode: the cache update folded into the Stage-1 launch (extra workgroups), or k_upd == null
  const void* k_upd; float* kbar_upd; int64_t ks_b, ks_h, ks_t;
  uint32_t* mask;
  int32_t* cnt;
  int32_t* idx;
  float* bias;
  float* tau;
  int batch, h_q, h_kv, g_q, n_q, n_kv, block, t_c, t_all, words, pos0, causal, window, ld;
  const int32_t* seq_lens;   // decode with per-sequence lengths (device, [batch]) or null
  int tok_base, tok_end;     // this launch covers query tokens [tok_base, tok_end) of every sequence
  int64_t qs_b, qs_h, qs_t;
  float xscale, pexp, alpha, inv_sigma;
};

enum { MODE_P1 = 0, MODE_P2 = 1, MODE_P4 = 2, MODE_GEN = 3, MODE_BISECT = 4 };
__host__ __device__ inline int s1_mode(float pexp) {
  if (pexp < 1.f) return MODE_BISECT;
  if (pexp == 1.f) return MODE_P1;
  if (pexp == 2.f) return MODE_P2;
  return pexp == 4.f ? MODE_P4 : MODE_GEN;
}

// u^p and u^(p-1) for u >= 0 (0 -> 0, and 0 for the derivative term as well)
template <int MODE>
__device__ __forceinline__ void pow_terms(float u, float p, float& f, float& g) {
  if constexpr (MODE == MODE_P1) {
    f = u; g = u > 0.f ? 1.f : 0.f;
  } else if constexpr (MODE == MODE_P2) {
    f = u * u; g = u;
  } else if constexpr (MODE == MODE_P4) {
    const float u2 = u * u; g = u2 * u; f = u2 * u2;
  } else {
    g = u > 0.f ? exp2f((p - 1.f) * log2f(u)) : 0.f;
    f = g * u;
  }
}
template <int MODE> __device__ __forceinline__ float pow_p(float u, float p) {
  float f, g; pow_terms<MODE>(u, p, f, g); return f;
}

// Reductions of four score rows at once that leave score row m % 4 in lane m of a DPP row (a
// quarter of the lanes each, all with the same bits): the order of the additions is that of
// row16_reduce.
__device__ __forceinline__ float add_quads(float x) {      // + the same score row's sums of the other three quads
  x += dpp_f<0x141>(dpp_f<0x1B>(x));                       // quad reversed, half row mirrored: lane m ^ 4
  return x + dpp_f<0x128>(x);                              // row_ror 8
}
// The values go through empty assembly: of plain selects over four copies of an array the compiler makes an indexed
// load, and puts the array into scratch memory for it (32 bytes a lane; a store and a dependent load between the row maxima
// and the first step of every solve: routing 8 heads x 300 tokens 12.6 us with, 12.1 without, 2 x 16 / 4 heads x 3001 tokens of
// d 64 19.8 -> 19.1; a decode step of 24 sequences of 32768 tokens, 32 / 2 heads, lists not asked for, 48.8 -> 48.3; same bits).
__device__ __forceinline__ float pick4(const float (&a)[4], int m) {
  float a0 = a[0], a1 = a[1], a2 = a[2], a3 = a[3];
  asm("" : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3));
  const float x = m & 1 ? a1 : a0, y = m & 1 ? a3 : a2;
  return m & 2 ? y : x;
}
__device__ __forceinline__ float sum4_scatter(const float (&a)[4], int m) {
  const float x = (m & 1 ? a[1] : a[0]) + dpp_f<0xB1>(m & 1 ? a[0] : a[1]);
  const float y = (m & 1 ? a[3] : a[2]) + dpp_f<0xB1>(m & 1 ? a[2] : a[3]);
  return add_quads((m & 2 ? y : x) + dpp_f<0x4E>(m & 2 ? x : y));
}
// lane m's four values of score rows 0..3 -> the four lanes' of its quad of score row m % 4
__device__ __forceinline__ void quad_transpose(const float (&a)[4], float (&t)[4], int m) {
  const float g0 = dpp_f<0xB1>(m & 1 ? a[0] : a[1]), g1 = dpp_f<0xB1>(m & 1 ? a[2] : a[3]);
  const float b0 = m & 1 ? g0 : a[0], b1 = m & 1 ? a[1] : g0, c0 = m & 1 ? g1 : a[2], c1 = m & 1 ? a[3] : g1;
  const float h0 = dpp_f<0x4E>(m & 2 ? b0 : c0), h1 = dpp_f<0x4E>(m & 2 ? b1 : c1);
  t[0] = m & 2 ? h0 : b0; t[1] = m & 2 ? h1 : b1; t[2] = m & 2 ? c0 : h0; t[3] = m & 2 ? c1 : h1;
}

// One bracketed Newton step of row state (tau, lo, hi, done) from the sums F = sum u^p,
// G = sum u^(p-1) at tau: without branches, each lane for the row it has (fp32 routing, one head of 1024 tokens, against
// branches: 15.4 -> 14.6 us, 8 / 2 heads x 4096 46.6 -> 45.0, at alpha 3 70.4 -> 68.5; same bits).
template <int MODE>
__device__ __forceinline__ void newton_step(float F, float G, float p, int n_cand, float& tau, float& lo, float& hi,
                                            bool& done) {
  const float f = F - 1.f;
  const float l = f > 0.f ? tau : lo, h = f > 0.f ? hi : tau, mid = 0.5f * (l + h);
  float cand = (MODE == MODE_BISECT || !(G > 0.f)) ? mid : tau + f / (p * G);
  // the root, or a Newton step below the fp32 spacing of tau
  const bool stay = f == 0.f || (MODE != MODE_BISECT && cand == tau);
  if (!(cand > l && cand < h)) cand = mid;
  const bool closed = !(cand > l && cand < h);               // bracket closed
  // alpha = 1.5: a Newton step s from the left leaves an error of about (k / 2G) s^2 <= (n / 2G) s^2
  // for k chunks in the support (f'' = 2k, f' = -2G); once that is below 2e-8 the step is final and the confirming
  // evaluation is skipped
  const float st = cand - tau;
  const bool last = MODE == MODE_P2 && f > 0.f && cand != mid && (float)n_cand * st * st < 4e-8f * G;
  const float next = closed ? l : cand;
  tau = done || stay ? tau : next;
  lo = l;
  hi = h;
  done = done || stay || closed || last;
}

// The register-resident Stage 1 (stage1_regs.hip), one object file per GQA group size.
hipError_t launch_s1_regs_g1(const S1Args& a, int head_dim, int mode, int max_cand, hipStream_t st);
hipError_t launch_s1_regs_g2(const S1Args& a, int head_dim, int mode, int max_cand, hipStream_t st);
hipError_t launch_s1_regs_g4(const S1Args& a, int head_dim, int mode, int max_cand, hipStream_t st);
hipError_t launch_s1_regs_g8(const S1Args& a, int head_dim, int mode, int max_cand, hipStream_t st);
hipError_t launch_s1_regs_g16(const S1Args& a, int head_dim, int mode, int max_cand, hipStream_t st);

}  // namespace dash
