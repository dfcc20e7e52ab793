// Backward, key side (bf16): dK, dV per 128-key tile, and the gradient of the chunk summaries.
// The chain is in backward.hip.
//
// bwd_kv_kernel.  A workgroup (4 waves) owns 128 keys, wave w the 32 keys 32 w .. + 31, and walks
// the 32-row tiles (32 / g_q tokens x g_q heads) that attend one of its chunks, found in the
// column masks.  Per step and wave: S = Q K^T, dP = dO V^T (rows x keys, K a register operand),
// P and dS = P (dP - D) in place, dV^T += dO^T P, dK^T += Q^T dS: 32 MFMAs, their operands 40 KB
// of LDS reads.  A wave accumulates all its rows itself, so nothing is exchanged at the end.
// The Q and dO rows of the next step are copied global -> LDS (two stages) while the current
// one is computed, one copy instruction at a time between the MFMAs, and its per-row scalars
// (mask bit, bias, log-sum-exp, D) are fetched into registers; one barrier per step.  The step is written
// slot by slot (one MFMA each) with the vector work of the softmax behind the MFMAs of the next
// product: the P of a step behind dP, its dS behind dV.
// What bounds it: the LDS pipe (40 KB per 32 MFMAs and wave: 1.25 of what 128 B/clk feeds) and
// the matrix pipe, two workgroups (two waves per SIMD) per CU, three at d = 64.  Measured on the training-shaped
// workload (4 x 16 heads x 8192 tokens): 3.85 ms with 64 keys per workgroup, both operands of S and dP
// in LDS, one tile buffer and dkbar in the same kernel -> 2.43 ms + 0.17 ms for dkbar; 2 x 16 / 4 heads x
// 3001 tokens, d 64 (192 key tiles, cut into parts): 375 -> 189 + 17 + 11 us.  Then, bwd_kv_kernel alone, both builds in
// turn: 2403 -> 2251 and 186 -> 168 us with the column masks' words loaded 32 row tiles ahead (two loads behind the barrier were
// waited for), the rows' scalars at 32-bit offsets, and no division per step.
//
// A launch with few key tiles cuts the row tiles of each into parts: fp32 partial sums go to the
// workspace and bwd_kv_reduce_kernel adds them in a fixed order.
//
// bwd_kbar_kernel: dkbar_c = xscale sum_rows dx q, a product over all (token, head) rows that
// have the chunk among their candidates (fp32 matrix cores, layout of f32_tiles.h).
#include <math.h>

#include "backward_args.h"
#include "bwd_tiles.h"
#include "dash_internal.h"
#include "f32_tiles.h"

namespace dash {

// number of parts of a key tile whose rows are nT 32-row tiles
__host__ __device__ inline int kv_parts(int nT, int steps_per_part) { return nT <= steps_per_part ? 1 : (nT + steps_per_part - 1) / steps_per_part; }

// The parts of a summary's gradient at p0, added in order; all loads in flight together.
constexpr int kMaxKbarParts = 16;
template <typename V> __device__ __forceinline__ V kbar_sum(const BwdArgs& a, const float* p0) {
  V x[kMaxKbarParts], sum = V{};
#pragma unroll
  for (int p = 0; p < kMaxKbarParts; p++) x[p] = p < a.kb_parts ? *reinterpret_cast<const V*>(p0 + p * a.kb_stride) : V{};
#pragma unroll
  for (int p = 0; p < kMaxKbarParts; p++) sum += x[p];
  return sum;
}

// TAIL: several heads and a last row tile that is not full.  The rows behind its last token are then copied as
// zeros: the buffer resources reach over what lies between the heads (the padding of a larger buffer, another
// head's rows), and 0 times what it holds could be a NaN.  In every launch the selection costs 0.5 % at d = 128
// (8.04 against 8.00 ms, forward and backward of the shape above), nothing at d = 64, where there is no other build.  No vector register is spilled, 14 to 16
// scalar ones are, to lanes of one.
// At d = 64 three waves per SIMD (168 registers, operands read one step ahead instead of two; the build without the selection would spill
// six): 2 x 16 / 4 heads x 3001 tokens 441 -> 408 us, forward and backward, 16 / 4 heads x 8000 1193 -> 1099, 8 heads x 4000 323 -> 309.
template <int D, bool TAIL>
__global__ __launch_bounds__(256, D == 64 ? 3 : 2) void bwd_kv_kernel(BwdArgs a) {
  using C = BCfg<D>;
  constexpr int RB = C::ROW_BYTES, HALF = 32 * RB, STAGE = 2 * HALF;   // a stage: 32 Q rows, 32 dO rows
  constexpr int KS = D / 16, NDT = C::NDT, RPI = 64 / C::NCH;         // RPI: rows per copy instruction of a wave
  constexpr int CP = 32 / (4 * RPI);                                  // copy instructions per wave, tensor and step
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  char* v_t = lds;                                  // 128 value rows
  char* ring = lds + 128 * RB;
  float* scal = reinterpret_cast<float*>(ring + 2 * STAGE);            // [4 waves][2][32]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int hbi = blockIdx.x % a.hb;
  const int ktile = blockIdx.x / a.hb, part = blockIdx.y;     // early key tiles (the most rows) first
  const int r = hbi % a.h_kv, b = hbi / a.h_kv;
  const int kpos0 = ktile * 128, my_key = kpos0 + wave * 32 + n;
  const int tokw = 32 / a.g_q;                      // tokens per 32-row tile
  const int g_log = 31 - __builtin_clz(a.g_q);
  const int n_T = (a.n_q + tokw - 1) / tokw;
  const int T_first = a.causal ? kpos0 / tokw : 0;
  const int parts = kv_parts(n_T - T_first, a.kv_steps);
  if (part >= parts) return;
  const int per = (n_T - T_first + parts - 1) / parts;
  const int T_beg = T_first + part * per, T_end = min(T_beg + per, n_T);
  const int c0 = kpos0 / a.block, c1 = kpos0 + 64 < a.n_kv ? (kpos0 + 64) / a.block : c0;
  const int c = wave < 2 ? c0 : c1;                 // this wave's chunk
  const bool wave_ok = kpos0 + wave * 32 < a.n_kv;

  // ---- the value rows into LDS, the key rows into registers ---------------------------------
  const u32x4 v_rs = make_rsrc(a.v + b * a.vs_b + r * a.vs_h, (((int64_t)a.n_kv - 1) * a.vs_t + D) * 2);
  const u32x4 q_rs = make_rsrc(a.q + b * a.qs_b + (int64_t)r * a.g_q * a.qs_h,
                               ((int64_t)(a.g_q - 1) * a.qs_h + ((int64_t)a.n_q - 1) * a.qs_t + D) * 2);
  const u32x4 o_rs = make_rsrc(a.d_o + b * a.os_b + (int64_t)r * a.g_q * a.os_h,
                               ((int64_t)(a.g_q - 1) * a.os_h + ((int64_t)a.n_q - 1) * a.os_t + D) * 2);
  const uint32_t lds0 = lds_addr_of(lds);
  const int c_row = wave * RPI + lane / C::NCH;     // tile row of copy instruction 0 (instruction i: + 4 RPI i)
  const uint32_t c_chunk = (uint32_t)(((lane % C::NCH) ^ swz<D>(c_row)) << 4);
  {
    const uint32_t v_off = (uint32_t)(c_row * (int)a.vs_t * 2) + c_chunk;
#pragma unroll
    for (int i = 0; i < 4 * CP; i++)
      copy16_to_lds(v_rs, lds0 + (i * 4 + wave) * 1024, v_off, (uint32_t)(kpos0 + i * 4 * RPI) * (uint32_t)a.vs_t * 2u);
  }
  bf16x8 kf[KS];
  {
    const uint16_t* kp = a.k + b * a.ks_b + r * a.ks_h + (int64_t)min(my_key, a.n_kv - 1) * a.ks_t + h * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) kf[ks] = *reinterpret_cast<const bf16x8*>(kp + ks * 16);
#pragma unroll
    for (int ks = 0; ks < KS; ks++) asm volatile("" : "+v"(kf[ks]));
  }
  const uint32_t q_off = (uint32_t)(((c_row / a.g_q) * (int)a.qs_t + (c_row % a.g_q) * (int)a.qs_h) * 2) + c_chunk;
  const uint32_t o_off = (uint32_t)(((c_row / a.g_q) * (int)a.os_t + (c_row % a.g_q) * (int)a.os_h) * 2) + c_chunk;
  const uint32_t q_step = (uint32_t)((4 * RPI / a.g_q) * (int)a.qs_t * 2), o_step = (uint32_t)((4 * RPI / a.g_q) * (int)a.os_t * 2);
  uint32_t cp_q = 0, cp_o = 0, cp_dst = 0;          // scalar offsets and LDS address of the step being copied
  int cp_left = 0;                                  // TAIL: its tokens before the end of the sequence
  auto copy_begin = [&](int T, int slot) {
    cp_q = (uint32_t)(T * tokw) * (uint32_t)a.qs_t * 2u;
    cp_o = (uint32_t)(T * tokw) * (uint32_t)a.os_t * 2u;
    cp_dst = lds0 + 128 * RB + slot * STAGE + wave * 1024;
    if constexpr (TAIL) cp_left = a.n_q - T * tokw;
  };
  const int c_tok = c_row / a.g_q, t_step = 4 * RPI / a.g_q;   // tokens of a copy instruction, TAIL
  auto copy_one = [&](int i) {                      // i < CP: Q rows, then dO rows
    const int j = i < CP ? i : i - CP;
    uint32_t off = i < CP ? q_off : o_off;
    if constexpr (TAIL) off = c_tok + j * t_step < cp_left ? off : 0x80000000u;   // past the end of any buffer (less than 2^31): zeros
    if (i < CP) copy16_to_lds(q_rs, cp_dst + j * 4096, off, cp_q + j * q_step);
    else copy16_to_lds(o_rs, cp_dst + HALF + j * 4096, off, cp_o + j * o_step);
  };

  // ---- operand read offsets -------------------------------------------------------------------
  const uint32_t a_rd = tile_off<D>(n, 8 * h), v_rd = tile_off<D>(wave * 32 + n, 8 * h);
  const int s16 = lane & 15, a16 = (lane >> 4) & 1;
  const uint32_t t_lo = tile_off<D>(4 * h + (s16 >> 2), 16 * a16 + 4 * (s16 & 3));
  const uint32_t t_hi = tile_off<D>(8 + 4 * h + (s16 >> 2), 16 * a16 + 4 * (s16 & 3));

  f32x16 dkacc[NDT], dvacc[NDT];
#pragma unroll
  for (int t = 0; t < NDT; t++) { dkacc[t] = zero16(); dvacc[t] = zero16(); }

  // ---- steps: the row tiles of [T_beg, T_end) whose bit is set in a column mask of this tile ----
  const uint32_t* cm0 = a.colmask + ((int64_t)hbi * a.t_all + c0) * a.cwords;
  const uint32_t* cm1 = a.colmask + ((int64_t)hbi * a.t_all + c1) * a.cwords;
  int it_wi = (T_beg >> 5) - 1;
  uint32_t it_bits = 0u, it_own = 0u;               // it_own: the bits of this wave's chunk
  bool it_on = false;
  const int it_last = a.cwords - 1;
  uint32_t it_n0 = cm0[min(it_wi + 1, it_last)], it_n1 = cm1[min(it_wi + 1, it_last)];   // the words of the next 32 row tiles
  auto next_step = [&]() -> int {
    while (it_bits == 0u) {
      it_wi++;
      if (it_wi * 32 >= T_end) return -1;
      const uint32_t w0 = __builtin_amdgcn_readfirstlane(it_n0), w1 = __builtin_amdgcn_readfirstlane(it_n1);
      it_n0 = cm0[min(it_wi + 1, it_last)];
      it_n1 = cm1[min(it_wi + 1, it_last)];
      it_own = wave < 2 ? w0 : w1;
      it_bits = w0 | w1;
      if (it_wi * 32 < T_beg) it_bits &= ~0u << (T_beg & 31);
      if (it_wi * 32 + 32 > T_end) it_bits &= (1u << (T_end & 31)) - 1u;
    }
    const int i = __builtin_ctz(it_bits);
    it_bits &= it_bits - 1u;
    it_on = wave_ok && ((it_own >> i) & 1u);
    return it_wi * 32 + i;
  };
  // lane n < 32: row n's scalars of a step, fetched one step ahead
  uint32_t f_mask = 0u;
  float f_bias = 0.f, f_lse = 0.f, f_dsum = 0.f;
  int f_tok = 0;
  const uint32_t* s_mask = a.mask + (int64_t)hbi * a.n_q * a.words + (c >> 5);
  const float* s_bias = a.biasd + (int64_t)hbi * a.n_q * a.t_all + c;
  const float* s_lse = a.lse + ((int64_t)b * a.h_q + r * a.g_q) * a.n_q;
  const float* s_dsum = a.dsum + ((int64_t)b * a.h_q + r * a.g_q) * a.n_q;
  const uint32_t s_head = (uint32_t)((n % a.g_q) * a.n_q);
  const int tok_off = n / a.g_q, own0 = c * a.block;      // first token whose own chunk is c
  auto fetch = [&](int T) {
    f_tok = T * tokw + tok_off;
    const uint32_t tk = (uint32_t)min(f_tok, a.n_q - 1);         // < 2^18: at most 2^11 chunks of 2^7 keys, 2^6 words
    f_mask = s_mask[__umul24(tk, a.words)];
    f_bias = s_bias[__umul24(tk, a.t_all)];         // meaningful only where the mask bit is set
    f_lse = s_lse[s_head + tk];
    f_dsum = s_dsum[s_head + tk];
  };
  float* sc = scal + wave * 64;                     // this wave's [bias - log-sum-exp][32], [D][32]

  int T = next_step();
  bool on = it_on;
  if (T >= 0) {
    copy_begin(T, 0);
#pragma unroll
    for (int i = 0; i < 2 * CP; i++) copy_one(i);
    fetch(T);
  }
  int slot = 0;
  while (T >= 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this wave's copies of the step have landed
    asm volatile("" : "+v"(it_n0), "+v"(it_n1), "+v"(f_mask), "+v"(f_bias), "+v"(f_lse), "+v"(f_dsum));   // and its loads
    if (lane < 32) {
      const bool bit = f_tok < a.n_q && ((f_mask >> (c & 31)) & 1u);
      const bool isdiag = a.causal && (uint32_t)(f_tok - own0) < (uint32_t)a.block;
      // bias - log-sum-exp in base-2 units (-inf: the row does not attend the chunk)
      sc[n] = bit ? (isdiag ? 0.f : f_bias * kLog2e) - f_lse : -INFINITY;
      sc[32 + n] = f_dsum;
    }
    __syncthreads();                                // everybody's copies; the other stage is no longer read
    const int tok0 = T * tokw;
    const bool cur_on = on;
    T = next_step();
    on = it_on;
    const bool more = T >= 0;
    if (more) { copy_begin(T, slot ^ 1); fetch(T); }
    if (!cur_on) {
      if (more) {
#pragma unroll
        for (int i = 0; i < 2 * CP; i++) copy_one(i);
      }
      slot ^= 1;
      continue;
    }
    const char* q_t = ring + slot * STAGE;
    const char* d_t = q_t + HALF;
    slot ^= 1;
    uint32_t a_b = a_rd, v_b = v_rd, tl = t_lo, th = t_hi;
    // opaque here, so that the per-slice offsets are formed next to their use
    asm volatile("" : "+v"(a_b), "+v"(v_b), "+v"(tl), "+v"(th));
    constexpr int AH = D == 64 ? 1 : 2;
    f32x16 s, dp;
    bf16x8 qa[KS], oa[KS], va[KS];
#pragma unroll
    for (int i = 0; i < AH; i++) qa[i] = read_a<D>(q_t, a_b, 2 * i);
    // S = Q K^T
#pragma unroll
    for (int i = 0; i < KS; i++) {
      if (i + AH < KS) qa[i + AH] = read_a<D>(q_t, a_b, 2 * (i + AH));
      else { oa[i + AH - KS] = read_a<D>(d_t, a_b, 2 * (i + AH - KS)); va[i + AH - KS] = read_a<D>(v_t, v_b, 2 * (i + AH - KS)); }
      if ((i & 1) == 0 && (i >> 1) < 2 * CP && more) copy_one(i >> 1);
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qa[i], kf[i], i == 0 ? zero16() : s, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    // the key mask matters only where the rows' own chunk is this one, or at the end of the sequence
    if ((a.causal && tok0 + tokw > own0 && tok0 < own0 + a.block) || kpos0 + 128 > a.n_kv) {
      int row0 = 4 * h;
      // the rows' tokens are formed here: kept in 16 registers throughout they had the kernel spill (4 x 16 heads x 8192 tokens
      // 7260 -> 7150 us, forward and backward)
      asm volatile("" : "+v"(row0));
      const int before = a.causal ? my_key - tok0 : -1;
#pragma unroll
      for (int j = 0; j < 16; j++)
        s[j] = (before > (row0 + (j >> 2) * 8 + (j & 3)) >> g_log || my_key >= a.n_kv) ? -INFINITY : s[j];
    }
    u32x4 pp[2], pd[2];
    auto p_quad = [&](int q4) {                     // P of accumulator registers 4 q4 .. + 3, in place
      const f32x4 b4 = *reinterpret_cast<const f32x4*>(sc + 8 * q4 + 4 * h);
#pragma unroll
      for (int i = 0; i < 4; i++) s[q4 * 4 + i] = __builtin_amdgcn_exp2f(fmaf(s[q4 * 4 + i], a.c1, b4[i]));
      pp[q4 >> 1][(q4 & 1) * 2] = cvt_bf16x2(s[q4 * 4], s[q4 * 4 + 1]);
      pp[q4 >> 1][(q4 & 1) * 2 + 1] = cvt_bf16x2(s[q4 * 4 + 2], s[q4 * 4 + 3]);
    };
    auto d_quad = [&](int q4) {                     // dS = P (dP - D)
      const f32x4 d4 = *reinterpret_cast<const f32x4*>(sc + 32 + 8 * q4 + 4 * h);
      float z[4];
#pragma unroll
      for (int i = 0; i < 4; i++) z[i] = s[q4 * 4 + i] * (dp[q4 * 4 + i] - d4[i]);
      pd[q4 >> 1][(q4 & 1) * 2] = cvt_bf16x2(z[0], z[1]);
      pd[q4 >> 1][(q4 & 1) * 2 + 1] = cvt_bf16x2(z[2], z[3]);
    };
    // dP = dO V^T; the P of this step behind its MFMAs
    bf16x8 ta[2 * NDT];
#pragma unroll
    for (int i = 0; i < KS; i++) {
      if (i + AH < KS) { oa[i + AH] = read_a<D>(d_t, a_b, 2 * (i + AH)); va[i + AH] = read_a<D>(v_t, v_b, 2 * (i + AH)); }
      else ta[i + AH - KS] = read_t<D>(d_t, tl, th, (i + AH - KS) / NDT, (i + AH - KS) % NDT);
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(oa[i], va[i], i == 0 ? zero16() : dp, 0, 0, 0);
      if constexpr (KS == 8) { if (i & 1) p_quad(i >> 1); }
      else p_quad(i);
      __builtin_amdgcn_sched_barrier(0);
    }
    // dV^T += dO^T P; the dS of this step behind its MFMAs
    bf16x8 tb[2 * NDT];
#pragma unroll
    for (int i = 0; i < 2 * NDT; i++) {
      if (i + AH < 2 * NDT) ta[i + AH] = read_t<D>(d_t, tl, th, (i + AH) / NDT, (i + AH) % NDT);
      else tb[i + AH - 2 * NDT] = read_t<D>(q_t, tl, th, (i + AH - 2 * NDT) / NDT, (i + AH - 2 * NDT) % NDT);
      dvacc[i % NDT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ta[i], __builtin_bit_cast(bf16x8, pp[i / NDT]), dvacc[i % NDT], 0, 0, 0);
      if constexpr (NDT == 4) { if (i & 1) d_quad(i >> 1); }
      else d_quad(i);
      __builtin_amdgcn_sched_barrier(0);
    }
    // dK^T += Q^T dS
#pragma unroll
    for (int i = 0; i < 2 * NDT; i++) {
      if (i + AH < 2 * NDT) tb[i + AH] = read_t<D>(q_t, tl, th, (i + AH) / NDT, (i + AH) % NDT);
      dkacc[i % NDT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tb[i], __builtin_bit_cast(bf16x8, pd[i / NDT]), dkacc[i % NDT], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // a workgroup without any step: its value copies

  // ---- outputs ---------------------------------------------------------------------------------
  if (parts > 1) {
    float* pk = a.kv_part + (((int64_t)ktile * a.hb + hbi) * a.kv_max_parts + part) * (2 * 128 * D) + (wave * 32 + n) * D;
#pragma unroll
    for (int t = 0; t < NDT; t++)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        const int d0 = t * 32 + q4 * 8 + h * 4;
        *reinterpret_cast<f32x4*>(pk + d0) = f32x4{dkacc[t][q4 * 4], dkacc[t][q4 * 4 + 1], dkacc[t][q4 * 4 + 2], dkacc[t][q4 * 4 + 3]};
        *reinterpret_cast<f32x4*>(pk + 128 * D + d0) = f32x4{dvacc[t][q4 * 4], dvacc[t][q4 * 4 + 1], dvacc[t][q4 * 4 + 2], dvacc[t][q4 * 4 + 3]};
      }
    return;
  }
  // block-mean summaries: every key of a complete chunk receives 1/B of the chunk's dkbar, whose parts are added
  // up once per workgroup (key by key, one load after the other, it took 30 us at 16 parts)
  float* kbs = reinterpret_cast<float*>(lds);       // [2 chunks][D]
  if (!a.dkbar_out) {
    __syncthreads();                                // nobody reads the tiles any more
    for (int i = tid; i < 2 * D; i += 256) {
      const int cc = i < D ? c0 : c1;
      kbs[i] = cc < a.t_c ? kbar_sum<float>(a, a.dkbar + ((int64_t)hbi * a.t_c + cc) * D + i % D) / (float)a.block : 0.f;
    }
    __syncthreads();
  }
  if (my_key >= a.n_kv) return;
  const bool fold = c < a.t_c && !a.dkbar_out;
  uint16_t* dkp = a.dk + b * a.ks_b + r * a.ks_h + (int64_t)my_key * a.ks_t;
  uint16_t* dvp = a.dv + b * a.vs_b + r * a.vs_h + (int64_t)my_key * a.vs_t;
#pragma unroll
  for (int t = 0; t < NDT; t++)
#pragma unroll
    for (int q4 = 0; q4 < 4; q4++) {
      const int d0 = t * 32 + q4 * 8 + h * 4;
      f32x4 kg = {0.f, 0.f, 0.f, 0.f};
      if (fold) kg = *reinterpret_cast<const f32x4*>(kbs + (wave < 2 ? 0 : D) + d0);
      float kv[4];
#pragma unroll
      for (int i = 0; i < 4; i++) kv[i] = fmaf(dkacc[t][q4 * 4 + i], a.scale, kg[i]);
      uint2 w;
      w.x = cvt_bf16x2(kv[0], kv[1]); w.y = cvt_bf16x2(kv[2], kv[3]);
      *reinterpret_cast<uint2*>(dkp + d0) = w;
      w.x = cvt_bf16x2(dvacc[t][q4 * 4], dvacc[t][q4 * 4 + 1]); w.y = cvt_bf16x2(dvacc[t][q4 * 4 + 2], dvacc[t][q4 * 4 + 3]);
      *reinterpret_cast<uint2*>(dvp + d0) = w;
    }
}

// Sum of the parts of the key tiles that have several (blockIdx.x = 8 keys of a tile).
template <int D>
__global__ __launch_bounds__(256) void bwd_kv_reduce_kernel(BwdArgs a) {
  constexpr int G4 = D / 4, KPW = 256 / G4;         // threads per key, keys per workgroup
  const int kg = blockIdx.x % (128 / KPW);
  const int id = blockIdx.x / (128 / KPW), hbi = id % a.hb, ktile = id / a.hb;
  const int r = hbi % a.h_kv, b = hbi / a.h_kv;
  const int kl = kg * KPW + threadIdx.x / G4, d0 = (threadIdx.x % G4) * 4;
  const int key = ktile * 128 + kl, c = key / a.block;
  const int tokw = 32 / a.g_q, n_T = (a.n_q + tokw - 1) / tokw;
  const int parts = kv_parts(n_T - (a.causal ? ktile * 128 / tokw : 0), a.kv_steps);
  if (parts == 1 || key >= a.n_kv) return;
  const float* pk = a.kv_part + ((int64_t)ktile * a.hb + hbi) * a.kv_max_parts * (2 * 128 * D) + kl * D + d0;
  f32x4 dk = {0.f, 0.f, 0.f, 0.f}, dv = dk, kgr = dk;
#pragma unroll 4
  for (int p = 0; p < parts; p++) {
    dk += *reinterpret_cast<const f32x4*>(pk + (int64_t)p * (2 * 128 * D));
    dv += *reinterpret_cast<const f32x4*>(pk + (int64_t)p * (2 * 128 * D) + 128 * D);
  }
  if (c < a.t_c && !a.dkbar_out)
    kgr = kbar_sum<f32x4>(a, a.dkbar + ((int64_t)hbi * a.t_c + c) * D + d0) * (1.f / (float)a.block);
  float kv[4];
#pragma unroll
  for (int i = 0; i < 4; i++) kv[i] = fmaf(dk[i], a.scale, kgr[i]);
  uint2 w;
  w.x = cvt_bf16x2(kv[0], kv[1]); w.y = cvt_bf16x2(kv[2], kv[3]);
  *reinterpret_cast<uint2*>(a.dk + b * a.ks_b + r * a.ks_h + (int64_t)key * a.ks_t + d0) = w;
  w.x = cvt_bf16x2(dv[0], dv[1]); w.y = cvt_bf16x2(dv[2], dv[3]);
  *reinterpret_cast<uint2*>(a.dv + b * a.vs_b + r * a.vs_h + (int64_t)key * a.vs_t + d0) = w;
}

// dkbar of 16 chunks from one part of the rows.  Four waves deal the 16-row tiles among them; the
// routing kernel has written dx (zero where not routed) for all candidates of every row.
template <int D>
__global__ __launch_bounds__(256, 4) void bwd_kbar_kernel(BwdArgs a, float* out, int n_groups) {
  using C = F32Cfg<D>;
  __shared__ float red[4][16 * C::LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, hq = lane >> 4;
  const int hbi = blockIdx.x % a.hb, grp = blockIdx.x / a.hb, part = blockIdx.y;   // early chunks (the most rows) first
  const int r = hbi % a.h_kv, b = hbi / a.h_kv;
  const int c = min(grp * 16 + n, a.t_c - 1);
  const int tokt = 16 / a.g_q;
  const int n_R = (a.n_q + tokt - 1) / tokt;
  const int R_first = a.causal ? min((grp * 16 + 1 + a.window) * a.block, a.n_q) / tokt : 0;   // rows with the first chunk among their candidates
  const int per = (n_R - R_first + a.kb_parts - 1) / a.kb_parts;
  const int R0 = R_first + part * per, R1 = min(R0 + per, n_R);
  f32x4 acc[C::NS];
#pragma unroll
  for (int i = 0; i < C::NS; i++) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  const uint16_t* qb = a.q + b * a.qs_b + (int64_t)r * a.g_q * a.qs_h;
  const float* dxb = a.dxd + ((int64_t)b * a.h_q + r * a.g_q) * a.n_q * a.t_all + c;
  // The rows of a tile are loaded by every lane, whether they count or not (from inside the arrays), while the tile
  // before is multiplied; the register bound keeps one copy of the accumulators.  Against loads in front of their use, everything
  // else the same: 24000 tokens, 8 / 2 heads, d 64 and 128: 150 -> 117, 202 -> 177 us; 20001 tokens, 4 heads, d 128: 64 -> 63;
  // 2 x 16 / 4 heads x 3001 tokens, d 64: 16.8 -> 14.6; 4 x 16 heads x 8192 tokens, d 128 (near the rate of memory: each group of
  // chunks reads q again): 180 -> 179.
  struct Rows { uint2 q[4][C::NV]; float dx[4]; };
  auto load = [&](int R) -> Rows {
    Rows x;
#pragma unroll
    for (int t = 0; t < 4; t++) {
      const int row = 4 * hq + t, head = row % a.g_q;
      const int64_t tk = min(R * tokt + row / a.g_q, a.n_q - 1);
      x.dx[t] = dxb[(head * (int64_t)a.n_q + tk) * a.t_all];
#pragma unroll
      for (int nv = 0; nv < C::NV; nv++) x.q[t][nv] = *reinterpret_cast<const uint2*>(qb + head * a.qs_h + tk * a.qs_t + 64 * nv + 4 * n);
    }
    return x;
  };
  Rows nx;
  if (R0 + wave < R1) nx = load(R0 + wave);
  for (int R = R0 + wave; R < R1; R += 4) {
    const int tok0 = R * tokt;
    const int n_cand = a.causal ? max(tok0 / a.block - a.window, 0) : a.t_c;
    const Rows x = nx;
    if (R + 4 < R1) nx = load(R + 4);
#pragma unroll
    for (int t = 0; t < 4; t++) {
      f32x4 row[C::NV];
#pragma unroll
      for (int nv = 0; nv < C::NV; nv++)
        row[nv] = f32x4{bf16_lo(x.q[t][nv].x), bf16_hi(x.q[t][nv].x), bf16_lo(x.q[t][nv].y), bf16_hi(x.q[t][nv].y)};
      // not written where the chunk is no candidate
      const float dx = tok0 + (4 * hq + t) / a.g_q < a.n_q && grp * 16 + n < n_cand ? x.dx[t] : 0.f;
      mma_outer<D>(row, dx, acc);
    }
  }
  put_tile<D>(red[wave], n, hq, acc, a.xscale);
  __syncthreads();
  for (int i = tid; i < 16 * D; i += 256) {
    const int cl = i / D, d = i % D, cc = grp * 16 + cl;
    if (cc < a.t_c)
      out[part * a.kb_stride + ((int64_t)hbi * a.t_c + cc) * D + d] = (red[0][cl * C::LD + d] + red[1][cl * C::LD + d]) + (red[2][cl * C::LD + d] + red[3][cl * C::LD + d]);
  }
}

// parts of the summary gradient -> the caller's array
__global__ void bwd_kbar_sum_kernel(const float* parts, float* out, int n_parts, int64_t stride) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= stride) return;
  float v = 0.f;
  for (int p = 0; p < n_parts; p++) v += parts[p * stride + i];
  out[i] = v;
}

template <int D, bool TAIL> static hipError_t launch_kv(const BwdArgs& a, hipStream_t st) {
  constexpr size_t lds = (size_t)128 * BCfg<D>::ROW_BYTES + 2 * 64 * BCfg<D>::ROW_BYTES + 4 * 64 * 4;
  auto kern = bwd_kv_kernel<D, TAIL>;
  static LdsOptIn opt_in;
  if (hipError_t e = allow_dyn_lds((const void*)kern, lds, opt_in); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)((a.n_kv + 127) / 128 * a.hb), (unsigned)a.kv_max_parts), dim3(256), lds, st, a);
  return hipGetLastError();
}

template <int D> static hipError_t launch_t(const BwdArgs& a, hipStream_t st) {
  hipError_t e;
  if (a.t_c > 0) {
    const int groups = (a.t_c + 15) / 16;
    float* out = a.dkbar_out && a.kb_parts == 1 ? a.dkbar_out : a.dkbar;
    hipLaunchKernelGGL(bwd_kbar_kernel<D>, dim3((unsigned)(groups * a.hb), (unsigned)a.kb_parts), dim3(256), 0, st, a, out, groups);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (a.dkbar_out && a.kb_parts > 1) {
      hipLaunchKernelGGL(bwd_kbar_sum_kernel, dim3((unsigned)((a.kb_stride + 255) / 256)), dim3(256), 0, st, a.dkbar, a.dkbar_out, a.kb_parts, a.kb_stride);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  const bool tail = a.g_q > 1 && a.n_q % (32 / a.g_q) != 0;
  if constexpr (D == 64) e = launch_kv<D, true>(a, st);
  else e = tail ? launch_kv<D, true>(a, st) : launch_kv<D, false>(a, st);
  if (e != hipSuccess) return e;
  if (a.kv_max_parts > 1) {
    const int ktiles = (a.n_kv + 127) / 128;
    hipLaunchKernelGGL(bwd_kv_reduce_kernel<D>, dim3((unsigned)(ktiles * a.hb * (128 * (D / 4) / 256))), dim3(256), 0, st, a);
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_bwd_kv(const BwdArgs& a, int head_dim, hipStream_t st) {
  return head_dim == 128 ? launch_t<128>(a, st) : launch_t<64>(a, st);
}

// How the key side is cut.  512 workgroups are resident (two per CU); a launch of fewer key tiles than
// that cuts each into parts of equal numbers of row tiles so that about 512 workgroups result (at
// least 8 steps each).  The summary gradient: about 1024 workgroups of 16 chunks.
void bwd_kv_plan(BwdArgs& a) {
  const int ktiles = (a.n_kv + 127) / 128, tokw = 32 / a.g_q, n_T = (a.n_q + tokw - 1) / tokw;
  a.kv_steps = n_T;
  a.kv_max_parts = 1;
  if ((int64_t)ktiles * a.hb < 512) {
    int64_t total = 0;
    for (int t = 0; t < ktiles; t++) total += n_T - (a.causal ? t * 128 / tokw : 0);
    const int64_t want = (total * a.hb + 511) / 512;
    a.kv_steps = want < 8 ? 8 : (int)want;
    a.kv_max_parts = kv_parts(n_T, a.kv_steps);
  }
  const int64_t groups = (int64_t)((a.t_c + 15) / 16) * a.hb;
  const int64_t p = groups > 0 ? 1024 / groups : 1;
  a.kb_parts = p < 1 ? 1 : (p > kMaxKbarParts ? kMaxKbarParts : (int)p);
  a.kb_stride = (int64_t)a.hb * a.t_c;      // x head_dim, set by the caller
}

}  // namespace dash
