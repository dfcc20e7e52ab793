// Backward pass of the prefill path (bf16 tensors; fp32 tensors: attn_f32.hip): gradients of the block-sparse
// attention with the routing prior with respect to q, k and v, including the
// path through the bias into the Stage-1 entmax weights and from there into the
// block-mean summaries (end of Sec. 3.3: the output is differentiable in q, k, v
// and the prior, so the gradient reaches Stage 1 and Stage 0; Sec. 3.5: the
// backward pass reuses the forward's chunk mask because the entmax Jacobian is
// zero outside the support).
//
// With P = softmax(z + d) over the attended tokens (z = q.k scale, d the bias
// of the token's chunk, 0 on the local chunks), o = P V and upstream dO:
//   dP = V dO,  D = <P, dP> (= <dO, o>),  dz = P (dP - D)
//   dq = scale K^T dz,  dK = scale dz q^T,  dV = P dO^T
//   dd_c = sum over the group's heads and the chunk's tokens of dz
//   dlnw_c = (dd_c - mean_R dd) / sigma,  dw_c = dlnw_c / w_c,  dw_hat = dw / g_q
//   dx_{h,c} = g_{h,c} (dw_hat_c - sum_j g_{h,j} dw_hat_j / sum_j g_{h,j}),
//       g_{h,c} = p u^(p-1) on the head's support, u = x - tau, p = 1/(alpha-1)
//   dq_h += c sum_c dx_{h,c} kbar_c,  dkbar_c = c sum_{rows} dx q,  c = gamma (alpha-1) scale
//   dK_j += dkbar_c / B for the keys of a complete chunk c (block mean).
//
// Kernels:
//   bwd_q_kernel   owns 128 (token, head) rows like the forward kernel and walks the
//                  union of their chunks; launched twice: <GRAD = false> for the row
//                  log-sum-exp and D, <GRAD = true> for dq (attention part, fp32), dd
//                  and a dense copy of the bias; the latter also marks, per chunk,
//                  which row tiles attend it.
//   bwd_route_kernel  (bwd_route.hip) 16 (token, head) rows per wave: prior and entmax
//                  Jacobian, dx per head and chunk, the routing part of dq, final dq.
//   bwd_kbar_kernel, bwd_kv_kernel  (bwd_kv.hip) the summaries' gradient; dK, dV of 128-key tiles
//                  over the row tiles that attend their chunks, without atomics.
//   bwd_f32_*      (attn_f32.hip) the same chain for fp32 tensors, with the routing kernel above.
// MFMA operand layouts are those of the forward kernel: every product is
// arranged so that the accumulator of the first product is directly the
// B operand of the second; the transposed operand comes from LDS through the
// transposing read.
#include <math.h>
#include <stdlib.h>

#include <type_traits>

#include "backward_args.h"
#include "bwd_tiles.h"
#include "common.h"
#include "dash_internal.h"
#include "lds_copy.h"

namespace dash {

// ---------------------------------------------------------------------------
// Row-owner kernel.
// ---------------------------------------------------------------------------
// GRAD = false: the first walk (row log-sum-exp and D into the workspace); GRAD = true: the second
// (dq, bias gradient, column masks).  Both walk like the forward kernel (stage2.hip): two-stage K and V
// rings filled by direct copies issued between the MFMAs of the tile before, one barrier per
// tile, q and dO fragments in registers, two workgroups per CU, and the tile written slot by slot with
// the vector work of one 32-key half behind the MFMAs of the next product.
// What bounds it: the matrix and LDS pipes about equally (48 KB of operand reads per 48 MFMAs and
// wave in the second walk).  Training-shaped workload (4 x 16 heads x 8192 tokens): 1.35 + 2.43 ms
// with a single tile buffer (copy, wait, compute) and dO as an LDS operand -> 1.30 + 2.07 ms; then, both builds in turn,
// 1266 -> 1184 and 2096 -> 2017 us (2 x 16 heads x 3001 tokens, d 64: 69 -> 64 and 107 -> 103) without the waits for the bias
// just asked for and for the bias gradient just stored; then 1184 -> 1148 and 2015 -> 1929 (65 -> 59 and 104 -> 96.5) with the tiles
// listed in front of the walk and a chunk's bias ready before the barrier, in every lane of its token.
template <int D, bool GRAD>
__global__ __launch_bounds__(256, 2) void bwd_q_kernel(BwdArgs a) {
  using C = BCfg<D>;
  constexpr int KS = D / 16, NDT = C::NDT;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  uint32_t* wgmask = reinterpret_cast<uint32_t*>(lds + 4 * C::TILE_BYTES);   // [64], after the K ring [2] and the V ring [2]
  uint32_t* wvmask = wgmask + 64;                                            // [4][64]
  uint16_t* list = reinterpret_cast<uint16_t*>(wgmask + 5 * 64);             // [4096]: the workgroup's tiles

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int hbi = blockIdx.x % a.hb;
  const int tile = a.n_tiles - 1 - blockIdx.x / a.hb;
  const int r = hbi % a.h_kv, b = hbi / a.h_kv;
  const int tokw = 32 / a.g_q;
  const int tok_w0 = tile * 4 * tokw + wave * tokw;
  const int sub_log = a.block >> 7;                     // log2 of the 64-key tiles of a chunk

  // the column masks that the second walk sets bits of: cleared by the first (a launch of its own took 4-5 us)
  if constexpr (!GRAD) {
    const int64_t words = (int64_t)a.hb * a.t_all * a.cwords;
    for (int64_t i = (int64_t)blockIdx.x * 256 + tid; i < words; i += (int64_t)gridDim.x * 256) a.colmask[i] = 0u;
  }

  const int my_tok = tok_w0 + n / a.g_q;
  const int my_head = r * a.g_q + n % a.g_q;
  const bool row_ok = my_tok < a.n_q;
  const int row_tok = row_ok ? my_tok : a.n_q - 1;
  const int row_pos = row_tok;                                   // n_q == n_kv
  const int cw = (tok_w0 < a.n_q ? tok_w0 : a.n_q - 1) / a.block;
  const bool wave_ok = tok_w0 < a.n_q;

  // ---- row fragments (B operands), complete before the tile loop -----------------
  bf16x8 qf[KS], dof[KS];
  {
    const uint16_t* qp = a.q + b * a.qs_b + my_head * a.qs_h + (int64_t)row_tok * a.qs_t + h * 8;
    const uint16_t* dop = a.d_o + b * a.os_b + my_head * a.os_h + (int64_t)row_tok * a.os_t + h * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) qf[ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 16);
#pragma unroll
    for (int ks = 0; ks < KS; ks++) dof[ks] = *reinterpret_cast<const bf16x8*>(dop + ks * 16);
  }

  // ---- chunk bitmaps ---------------------------------------------------------
  // Every lane tracks the token of its row, as in s2_attend_kernel; the first of a token's lanes writes what is the token's.
  const int64_t trk_base = ((int64_t)b * a.h_kv + r) * a.n_q + min(tok_w0, a.n_q - 1);   // uniform; a lane's row by offset
  const uint32_t* trk_mask = a.mask + trk_base * a.words;
  const __amdgpu_buffer_rsrc_t trk_bias = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(a.bias) + trk_base * a.t_all, 0, max(min(tokw, a.n_q - tok_w0), 0) * a.t_all * 4, 0x00020000);
  auto ask_bias = [&](uint32_t at) -> float { return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(trk_bias, at, 0, 0)); };
  const uint32_t trk_m0 = row_ok ? (uint32_t)(n / a.g_q * a.words) : 0u, trk_b0 = row_ok ? (uint32_t)(n / a.g_q * a.t_all) : 0u;
  uint32_t trk_at = row_ok ? trk_b0 * 4u : ~3u, trk_word = 0;
  const bool trk_lead = h == 0 && n % a.g_q == 0;
  bool trk_has = false;
  float trk_old = 0.f, trk_next = ask_bias(trk_at);

  for (int i = tid; i < 5 * 64; i += 256) wgmask[i] = 0u;
  __syncthreads();
  if (wave_ok)
    or_mask_rows(a.mask + (((int64_t)b * a.h_kv + r) * a.n_q + tok_w0) * a.words, min(tokw, a.n_q - tok_w0) * a.words,
                 a.words, wvmask + wave * 64, wgmask, lane);
  __syncthreads();
  // tell the key side which chunks this wave's 32-row tile attends
  if constexpr (GRAD)
  if (wave_ok)
    for (int wi = lane; wi < a.words; wi += 64) {
      uint32_t m = wvmask[wave * 64 + wi];
      const int T = tile * 4 + wave;
      while (m) {
        const int c = wi * 32 + __builtin_ctz(m);
        m &= m - 1u;
        if (c < a.t_all) atomicOr(&a.colmask[((int64_t)hbi * a.t_all + c) * a.cwords + (T >> 5)], 1u << (T & 31));
      }
    }

  const int n_it = list_tiles<256>(wgmask, wvmask, list, sub_log, tid) << sub_log;
  __syncthreads();
  auto entry = [&](int i) -> int { return list[max(min(i, n_it - 1), 0)]; };   // behind the last tile: that one again
  int e_cur = __builtin_amdgcn_readfirstlane(entry(0)), e_next = __builtin_amdgcn_readfirstlane(entry(1)), e_ahead = 0;
  if (n_it == 0) e_cur = e_next = 0;             // no list: whatever lies there
  trk_word = trk_mask[trk_m0 + ((e_cur & 0xfff) >> sub_log >> 5)];

  // ---- tile copies -------------------------------------------------------------
  const u32x4 k_rs = make_rsrc(a.k + b * a.ks_b + r * a.ks_h, (((int64_t)a.n_kv - 1) * a.ks_t + D) * 2);
  const u32x4 v_rs = make_rsrc(a.v + b * a.vs_b + r * a.vs_h, (((int64_t)a.n_kv - 1) * a.vs_t + D) * 2);
  const uint32_t lds0 = lds_addr_of(lds);
  const int c_row = (wave * 64 + lane) / C::NCH, c_pos = lane % C::NCH;
  const uint32_t k_off = (uint32_t)(c_row * (int)a.ks_t * 2 + ((c_pos ^ swz<D>(c_row)) << 4));
  const uint32_t v_off = (uint32_t)(c_row * (int)a.vs_t * 2 + ((c_pos ^ swz<D>(c_row)) << 4));
  const uint32_t k_step = (uint32_t)(C::ROWS_PER_COPY * (int)a.ks_t * 2);
  const uint32_t v_step = (uint32_t)(C::ROWS_PER_COPY * (int)a.vs_t * 2);
  uint32_t cp_k = 0, cp_v = 0;   // scalar byte offsets of the tile being copied
  const uint32_t k_tile = (uint32_t)a.ks_t * 128u, v_tile = (uint32_t)a.vs_t * 128u;   // bytes from tile to tile
  auto copy_begin = [&](int t) { cp_k = (uint32_t)t * k_tile; cp_v = (uint32_t)t * v_tile; };
  auto copy_one = [&](int c, int slot) {
    if (c < C::COPIES)
      copy16_to_lds(k_rs, lds0 + slot * C::TILE_BYTES + wave * 1024 + c * 4096, k_off, cp_k + c * k_step);
    else
      copy16_to_lds(v_rs, lds0 + (2 + slot) * C::TILE_BYTES + wave * 1024 + (c - C::COPIES) * 4096, v_off,
                    cp_v + (c - C::COPIES) * v_step);
  };

  // ---- operand read offsets ------------------------------------------------------
  // A operand: lane (n, h) reads logical chunk 2 ks + h of rows n, 32 + n.
  // Transposing read: lanes 16 g' .. 16 g' + 15 serve d columns 16 (g' & 1) .. + 15
  // of a d-tile and contraction half h = g' >> 1; lane s of the group points at
  // tile row 4 h + s / 4 (+ 8 for the second read), d offset 16 (g' & 1) + 4 (s % 4).
  const uint32_t a_rd = tile_off<D>(n, 8 * h);
  const int s16 = lane & 15, a16 = (lane >> 4) & 1;
  const uint32_t t_lo = tile_off<D>(4 * h + (s16 >> 2), 16 * a16 + 4 * (s16 & 3));
  const uint32_t t_hi = tile_off<D>(8 + 4 * h + (s16 >> 2), 16 * a16 + 4 * (s16 & 3));

  // first walk: running max, sum of exponentials and sum of exponentials times dP; D =
  // <P, dP> = <dO, o> is taken from the latter two in fp32 (the stored bf16 output would
  // put its rounding error into every dz of the row).  Second walk: both come from the workspace.
  float m_run = -INFINITY, l_run = 0.f, dn_run = 0.f, lse2 = 0.f, dsum = 0.f, db_acc = 0.f;
  f32x16 dqacc[GRAD ? NDT : 1];
#pragma unroll
  for (int t = 0; t < (GRAD ? NDT : 1); t++) dqacc[t] = zero16();
  if constexpr (GRAD) {
    const int64_t row = ((int64_t)b * a.h_q + my_head) * a.n_q + row_tok;
    lse2 = a.lse[row];
    dsum = a.dsum[row];
    asm volatile("" : "+v"(lse2), "+v"(dsum));
  }
  float* biasd = a.biasd + trk_base * a.t_all;
  float* dbd = a.dbd + trk_base * a.t_all;
  float bias_row = 0.f;
  bool diag = false;
  auto begin_chunk = [&](int u) {
    trk_has = false;
    bias_row = 0.f;
    if (a.causal && u == cw) return;
    const bool bit = row_ok && ((trk_word >> (u & 31)) & 1u);
    const float next = trk_old + trk_next;   // one of them is 0
    bias_row = bit ? next * kLog2e : -INFINITY;
    if (GRAD) { if (bit && trk_lead) biasd[trk_b0 + u] = next; }
    trk_old = bit ? 0.f : next;
    trk_at += bit ? 4u : 0u;
    trk_next = ask_bias(bit ? trk_at : ~3u);   // by every lane: see s2_attend_kernel
    trk_has = bit;
  };

  // ---- one 64-key tile, in two 32-key halves -----------------------------------------
  auto tile_math = [&](auto p_tag, bool masked, int kpos0, bool more) {
    constexpr int P = decltype(p_tag)::value;
    const char* kb = lds + P * C::TILE_BYTES;
    const char* vb = lds + (2 + P) * C::TILE_BYTES;
    constexpr int AH = 2;
    f32x16 s[2], dp[2];
    // S^T = K Q^T or dP^T = V dO^T of half kt; after MFMA i: behind(i)
    auto product = [&](const char* t, const bf16x8 (&rows)[KS], int kt, auto&& behind) -> f32x16 {
      f32x16 acc;
      bf16x8 op[KS];
#pragma unroll
      for (int i = 0; i < AH; i++) op[i] = read_a<D>(t, a_rd, 2 * i + kt);
#pragma unroll
      for (int i = 0; i < KS; i++) {
        if (i + AH < KS) op[i + AH] = read_a<D>(t, a_rd, 2 * (i + AH) + kt);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[i], rows[i], i == 0 ? zero16() : acc, 0, 0, 0);
        behind(i);
        __builtin_amdgcn_sched_barrier(0);
      }
      return acc;
    };
    // quad index of slot i (four quads of 4 keys over KS slots)
    auto quad_at = [](int i) -> int { return KS == 8 ? ((i & 1) ? i >> 1 : -1) : i; };
    // key mask: causal inside the diagonal chunk, and the end of the sequence
    auto mask_half = [&](int kt) {
      if (masked) {
        const int k0 = kpos0 + 32 * kt + 4 * h;
        int lim = min(diag ? row_pos - k0 : 0x7fffffff, a.n_kv - 1 - k0);
        asm volatile("" : "+v"(lim));
#pragma unroll
        for (int j = 0; j < 16; j++) {
          const int c = (j >> 2) * 8 + (j & 3);
          s[kt][j] = c > lim ? -INFINITY : s[kt][j];
        }
      }
    };
    // the copies of the next tile, one per slot, starting at slot `i0` of the tile
    auto copies = [&](int i) {
      if (i < 2 * C::COPIES && more) copy_one(i, P ^ 1);
    };
    if constexpr (!GRAD) {
      s[0] = product(kb, qf, 0, [&](int i) { copies(i); });
      s[1] = product(kb, qf, 1, [&](int i) { copies(KS + i); });
      mask_half(0);
      mask_half(1);
      float mloc = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < 2; kt++)
#pragma unroll
        for (int j = 0; j < 16; j += 2) mloc = fmaxf(fmaxf(mloc, s[kt][j]), s[kt][j + 1]);
      mloc = fmaxf(mloc, __shfl_xor(mloc, 32));
      const float m_new = fmaxf(m_run, fmaf(mloc, a.c1, bias_row));
      const float m_use = m_new == -INFINITY ? 0.f : m_new;
      const float corr = __builtin_amdgcn_exp2f(m_run - m_use), off = bias_row - m_use;
      m_run = m_new;
      // The tile's sums first, then the running ones: D enters every dz of the row, and what it is off by
      // comes back, times 1 / w, where a chunk is next to its threshold.  (All keys in one chain: the bias
      // gradients of a row of 1152 keys, which cancel, add up to 1e-6 instead of 6e-8.)
      float l_tile = 0.f, dn_tile = 0.f;
      auto e_quad = [&](int kt, int q4) {
        if (q4 < 0) return;
#pragma unroll
        for (int j = 4 * q4; j < 4 * q4 + 4; j++) {
          s[kt][j] = __builtin_amdgcn_exp2f(fmaf(s[kt][j], a.c1, off));
          l_tile += s[kt][j];
        }
      };
      auto n_quad = [&](int kt, int q4) {
        if (q4 < 0) return;
#pragma unroll
        for (int j = 4 * q4; j < 4 * q4 + 4; j++) dn_tile = fmaf(s[kt][j], dp[kt][j], dn_tile);
      };
      dp[0] = product(vb, dof, 0, [&](int i) { e_quad(0, quad_at(i)); });
      dp[1] = product(vb, dof, 1, [&](int i) { e_quad(1, quad_at(i)); n_quad(0, quad_at(i)); });
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) n_quad(1, q4);
      l_run = fmaf(l_run, corr, l_tile);
      dn_run = fmaf(dn_run, corr, dn_tile);
    } else {
      const float off = bias_row - lse2;
      u32x4 pb[4];
      auto p_quad = [&](int kt, int q4) {
        if (q4 < 0) return;
#pragma unroll
        for (int j = 4 * q4; j < 4 * q4 + 4; j++) s[kt][j] = __builtin_amdgcn_exp2f(fmaf(s[kt][j], a.c1, off));
      };
      auto d_quad = [&](int kt, int q4) {     // dS^T = P^T (dP^T - D), packed as the B operand of the last product
        if (q4 < 0) return;
        float z[4];
#pragma unroll
        for (int i = 0; i < 4; i++) z[i] = s[kt][4 * q4 + i] * (dp[kt][4 * q4 + i] - dsum);
        db_acc += (z[0] + z[1]) + (z[2] + z[3]);
        pb[2 * kt + (q4 >> 1)][(q4 & 1) * 2] = cvt_bf16x2(z[0], z[1]);
        pb[2 * kt + (q4 >> 1)][(q4 & 1) * 2 + 1] = cvt_bf16x2(z[2], z[3]);
      };
      s[0] = product(kb, qf, 0, [&](int i) { copies(i); });
      mask_half(0);
      dp[0] = product(vb, dof, 0, [&](int i) { copies(KS + i); p_quad(0, quad_at(i)); });
      s[1] = product(kb, qf, 1, [&](int i) { d_quad(0, quad_at(i)); });
      mask_half(1);
      dp[1] = product(vb, dof, 1, [&](int i) { p_quad(1, quad_at(i)); });
      // dQ^T += K^T dS^T
      bf16x8 tr[4 * NDT];
#pragma unroll
      for (int i = 0; i < AH; i++) tr[i] = read_t<D>(kb, t_lo, t_hi, i / NDT, i % NDT);
#pragma unroll
      for (int i = 0; i < 4 * NDT; i++) {
        if (i + AH < 4 * NDT) tr[i + AH] = read_t<D>(kb, t_lo, t_hi, (i + AH) / NDT, (i + AH) % NDT);
        dqacc[i % NDT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr[i], __builtin_bit_cast(bf16x8, pb[i / NDT]), dqacc[i % NDT], 0, 0, 0);
        if (i < 2 * NDT) d_quad(1, NDT == 4 ? ((i & 1) ? i >> 1 : -1) : i);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  // ---- main loop: as in the forward kernel ------------------------------------------------
#pragma unroll
  for (int ks = 0; ks < KS; ks++) asm volatile("" : "+v"(qf[ks]), "+v"(dof[ks]));   // landed before the copies are in flight
  if (n_it > 0) {
    copy_begin(e_cur & 0xfff);
#pragma unroll
    for (int c = 0; c < 2 * C::COPIES; c++) copy_one(c, 0);
  }
  // the bias gradient of a chunk is stored behind the next wait for copies, which would be one for the store
  float db_out = 0.f;
  int db_u = -1;
  auto put_db = [&]() {
    if constexpr (GRAD) {
      if (db_u >= 0) dbd[trk_b0 + db_u] = db_out;
      db_u = -1;
    }
  };
  auto iteration = [&](auto p_tag, int it) {
    constexpr int P = decltype(p_tag)::value;
    const int t_cur = e_cur & 0xfff, t_next = e_next & 0xfff, u = t_cur >> sub_log, un = t_next >> sub_log;
    const bool on = (e_cur >> (12 + wave)) & 1, more = it + 1 < n_it;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's copies of the tile have landed, and its loads
    // whatever needs no tile stands before the barrier
    put_db();
    diag = a.causal && u == cw;
    if (on && (t_cur & sub_log) == 0) begin_chunk(u);
    if ((un ^ u) >> 5) trk_word = trk_mask[trk_m0 + (un >> 5)];   // arrives with the next tile's copies
    if (more) copy_begin(t_next);
    asm volatile("s_barrier" ::: "memory");
    e_ahead = entry(it + 2);
    if (on) {
      const int kpos0 = t_cur * 64;
      tile_math(p_tag, diag || kpos0 + 64 > a.n_kv, kpos0, more);
      if (GRAD && (t_cur & sub_log) == sub_log) {
        // bias gradient of chunk u: sum over the keys (both lane halves) and the token's heads (adjacent lanes)
        float tot = db_acc + __shfl_xor(db_acc, 32);
        for (int o = 1; o < a.g_q; o <<= 1) tot += __shfl_xor(tot, o);
        db_out = tot;
        db_u = trk_has && trk_lead ? u : -1;
        db_acc = 0.f;
      }
    } else if (more) {
#pragma unroll
      for (int c = 0; c < 2 * C::COPIES; c++) copy_one(c, P ^ 1);
    }
    e_cur = e_next;
    e_next = __builtin_amdgcn_readfirstlane(e_ahead);
  };
  for (int it = 0; it < n_it;) {
    iteration(std::integral_constant<int, 0>{}, it);
    if (++it >= n_it) break;
    iteration(std::integral_constant<int, 1>{}, it);
    ++it;
  }
  put_db();

  // ---- outputs -----------------------------------------------------------------
  const float l_tot = l_run + __shfl_xor(l_run, 32);
  const float dn_tot = dn_run + __shfl_xor(dn_run, 32);
  if (!row_ok) return;
  const int64_t row = ((int64_t)b * a.h_q + my_head) * a.n_q + my_tok;
  if constexpr (!GRAD) {
    if (h == 0) {
      a.lse[row] = (m_run == -INFINITY ? 0.f : m_run) + __builtin_amdgcn_logf(l_tot);   // v_log_f32: log2
      a.dsum[row] = l_tot > 0.f ? dn_tot / l_tot : 0.f;
    }
  } else {
    float* dq = a.dq32 + row * D;
#pragma unroll
    for (int t = 0; t < NDT; t++)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        const int m0 = q4 * 8 + h * 4;
        float4 w;
        w.x = dqacc[t][q4 * 4 + 0] * a.scale; w.y = dqacc[t][q4 * 4 + 1] * a.scale;
        w.z = dqacc[t][q4 * 4 + 2] * a.scale; w.w = dqacc[t][q4 * 4 + 3] * a.scale;
        *reinterpret_cast<float4*>(dq + t * 32 + m0) = w;
      }
  }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
static size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

// Carves the workspace (ws may be null: sizes only) and fills the sizes of the arguments.  Returns
// the bytes.
static size_t carve_workspace(BwdArgs& a, const dash_params& p, const Layout& L, char* ws) {
  a.h_q = p.h_q; a.h_kv = p.h_kv; a.g_q = L.g_q; a.n_q = p.n_q; a.n_kv = p.n_kv; a.block = p.block_size;
  a.t_c = L.t_c; a.t_all = L.t_all; a.words = L.words; a.causal = p.causal; a.window = p.window;
  a.hb = p.h_kv * p.batch;
  const int tok_tile = 4 * (32 / L.g_q);
  a.n_tiles = (p.n_q + tok_tile - 1) / tok_tile;
  a.cwords = (4 * a.n_tiles + 31) / 32;
  bwd_kv_plan(a);
  a.kb_stride *= p.head_dim;
  const size_t rows_q = (size_t)p.batch * p.h_q * p.n_q, rows_kv = (size_t)p.batch * p.h_kv * p.n_q;
  size_t off = 0;
  auto take = [&](size_t bytes) { char* q = ws ? ws + off : nullptr; off += al256(bytes); return q; };
  a.lse = (float*)take(rows_q * 4);
  a.dsum = (float*)take(rows_q * 4);
  a.biasd = (float*)take(rows_kv * L.t_all * 4);
  a.dbd = (float*)take(rows_kv * L.t_all * 4);
  a.dxd = (float*)take(rows_q * L.t_all * 4);
  a.dq32 = (float*)take(rows_q * p.head_dim * 4);
  a.colmask = (uint32_t*)take((size_t)a.hb * L.t_all * a.cwords * 4);
  a.dkbar = (float*)take((size_t)a.kb_parts * a.kb_stride * 4);
  a.kv_part = (float*)take(a.kv_max_parts > 1 ? (size_t)((p.n_kv + 127) / 128) * a.hb * a.kv_max_parts * 2 * 128 * p.head_dim * 4 : 0);
  return off;
}

size_t backward_workspace_bytes(const dash_params& p, const Layout& L) {
  BwdArgs a;
  return carve_workspace(a, p, L, nullptr);
}

template <int D> static hipError_t launch_bwd_f32(const BwdArgs& a, hipStream_t st) {
  hipError_t e;
  if ((e = launch_bwd_f32_rows(a, D, st)) != hipSuccess) return e;
  if ((e = launch_bwd_route(a, D, false, st)) != hipSuccess) return e;
  return launch_bwd_f32_keys(a, D, st);
}

template <int D> static hipError_t launch_bwd_t(const BwdArgs& a, hipStream_t st) {
  using C = BCfg<D>;
  static LdsOptIn done_lse, done_grad;
  hipError_t e;
  {
    const size_t lds = 4 * C::TILE_BYTES + 5 * 64 * 4 + 4096 * 2;
    auto kern = bwd_q_kernel<D, false>;
    if ((e = allow_dyn_lds((const void*)kern, lds, done_lse)) != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(a.n_tiles * a.hb), dim3(256), lds, st, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  {
    const size_t lds = 4 * C::TILE_BYTES + 5 * 64 * 4 + 4096 * 2;
    auto kern = bwd_q_kernel<D, true>;
    if ((e = allow_dyn_lds((const void*)kern, lds, done_grad)) != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(a.n_tiles * a.hb), dim3(256), lds, st, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if ((e = launch_bwd_route(a, D, true, st)) != hipSuccess) return e;
  return launch_bwd_kv(a, D, st);
}

hipError_t launch_backward(const dash_params& p, const Layout& L, const void* q, const void* k, const void* v,
                           const void* d_o, const float* kbar, const uint32_t* mask,
                           const float* bias, const float* tau, void* dq, void* dk, void* dv, float* dkbar_out,
                           char* ws, hipStream_t st) {
  BwdArgs a;
  a.dkbar_out = dkbar_out;
  a.q = (const uint16_t*)q; a.k = (const uint16_t*)k; a.v = (const uint16_t*)v;
  a.d_o = (const uint16_t*)d_o;
  a.dq = (uint16_t*)dq; a.dk = (uint16_t*)dk; a.dv = (uint16_t*)dv;
  a.kbar = kbar; a.mask = mask; a.bias = bias; a.tau = tau;
  carve_workspace(a, p, L, ws);
  a.qs_b = p.q_stride[0]; a.qs_h = p.q_stride[1]; a.qs_t = p.q_stride[2];
  a.ks_b = p.k_stride[0]; a.ks_h = p.k_stride[1]; a.ks_t = p.k_stride[2];
  a.vs_b = p.v_stride[0]; a.vs_h = p.v_stride[1]; a.vs_t = p.v_stride[2];
  a.os_b = p.o_stride[0]; a.os_h = p.o_stride[1]; a.os_t = p.o_stride[2];
  a.c1 = L.scale * kLog2e; a.scale = L.scale; a.xscale = L.xscale; a.pexp = L.pexp; a.sigma = p.sigma;
  if (p.dtype == DASH_F32)
    return p.head_dim == 128 ? launch_bwd_f32<128>(a, st) : launch_bwd_f32<64>(a, st);
  return p.head_dim == 128 ? launch_bwd_t<128>(a, st) : launch_bwd_t<64>(a, st);
}

}  // namespace dash
