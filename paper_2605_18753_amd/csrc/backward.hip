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

#include "backward_args.h"
#include "bwd_tiles.h"
#include "common.h"
#include "dash_internal.h"
#include "lds_copy.h"

namespace dash {

__global__ void bwd_fill_zero_kernel(uint32_t* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

// ---------------------------------------------------------------------------
// Row-owner kernel.
// ---------------------------------------------------------------------------
// GRAD = false: the first walk (row log-sum-exp and D into the workspace; few registers, dO
// fragments in registers, three workgroups per CU).  GRAD = true: the second walk (dq, bias
// gradient, column masks; dO rows as an LDS operand, two workgroups per CU).
template <int D, bool GRAD>
__global__ __launch_bounds__(256, GRAD ? 2 : 3) void bwd_q_kernel(BwdArgs a) {
  using C = BCfg<D>;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  char* k_t = lds;                            // K tile
  char* v_t = lds + C::TILE_BYTES;            // V tile
  char* do_t = lds + 2 * C::TILE_BYTES;       // GRAD: dO rows of the workgroup's 128 rows (stationary)
  uint32_t* wgmask = reinterpret_cast<uint32_t*>(lds + (GRAD ? 4 : 2) * C::TILE_BYTES);   // [64]
  uint32_t* wvmask = wgmask + 64;                                            // [4][64]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int hbi = blockIdx.x % a.hb;
  const int tile = a.n_tiles - 1 - blockIdx.x / a.hb;
  const int r = hbi % a.h_kv, b = hbi / a.h_kv;
  const int tokw = 32 / a.g_q;
  const int tok_w0 = tile * 4 * tokw + wave * tokw;
  const int nsub = a.block >> 6;

  const int my_tok = tok_w0 + n / a.g_q;
  const int my_head = r * a.g_q + n % a.g_q;
  const bool row_ok = my_tok < a.n_q;
  const int row_tok = row_ok ? my_tok : a.n_q - 1;
  const int row_pos = row_tok;                                   // n_q == n_kv
  const int cw = (tok_w0 < a.n_q ? tok_w0 : a.n_q - 1) / a.block;
  const bool wave_ok = tok_w0 < a.n_q;

  // ---- row fragments as B operands: q in registers; dO in registers (first walk) or in LDS
  // (second walk, each wave its own 32 rows)
  bf16x8 qf[D / 16], dof[GRAD ? 1 : D / 16];
  {
    const uint16_t* qp = a.q + b * a.qs_b + my_head * a.qs_h + (int64_t)row_tok * a.qs_t + h * 8;
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++) qf[ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 16);
  }
  if constexpr (!GRAD) {
    const uint16_t* dop = a.d_o + b * a.os_b + my_head * a.os_h + (int64_t)row_tok * a.os_t + h * 8;
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++) dof[ks] = *reinterpret_cast<const bf16x8*>(dop + ks * 16);
  } else {
    const u32x4 o_rs = make_rsrc(a.d_o + b * a.os_b + (int64_t)r * a.g_q * a.os_h,
                                 ((int64_t)(a.g_q - 1) * a.os_h + ((int64_t)a.n_q - 1) * a.os_t + D) * 2);
    constexpr int RPI = 64 / C::NCH;             // rows one copy instruction covers
#pragma unroll
    for (int i = 0; i < 32 / RPI; i++) {
      const int rw = i * RPI + lane / C::NCH;    // row of this wave
      const int tk = min(tok_w0 + rw / a.g_q, a.n_q - 1);
      const uint32_t voff = (uint32_t)((tk * (int)a.os_t + (rw % a.g_q) * (int)a.os_h) * 2) +
                            (uint32_t)(((lane % C::NCH) ^ swz<D>(wave * 32 + rw)) << 4);
      copy16_to_lds(o_rs, lds_addr_of(do_t) + (wave * 32 + i * RPI) * C::ROW_BYTES, voff, 0u);
    }
  }
  const uint32_t do_rd = tile_off<D>(wave * 32 + n, 8 * h);

  // ---- chunk bitmaps ---------------------------------------------------------
  const int trk_tok = tok_w0 + lane;
  const bool trk_ok = lane < tokw && trk_tok < a.n_q;
  const int64_t trk_base = ((int64_t)b * a.h_kv + r) * a.n_q + (trk_ok ? trk_tok : 0);
  const uint32_t* trk_mask = a.mask + trk_base * a.words;
  const float* trk_bias = a.bias + trk_base * a.t_all;
  int trk_rank = 0, trk_wi = -1;
  uint32_t trk_word = 0;
  bool trk_has = false;

  for (int i = tid; i < 5 * 64; i += 256) wgmask[i] = 0u;
  __syncthreads();
  if (wave_ok)
    for (int wi = lane; wi < a.words; wi += 64) {
      uint32_t m = 0u;
      for (int t = 0; t < tokw; t++)
        if (tok_w0 + t < a.n_q)
          m |= a.mask[(((int64_t)b * a.h_kv + r) * a.n_q + tok_w0 + t) * a.words + wi];
      wvmask[wave * 64 + wi] = m;
      if (m) atomicOr(&wgmask[wi], m);
    }
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

  // ---- tile iterator ---------------------------------------------------------
  int it_wi = -1, it_sub = nsub - 1, it_u = -1;
  uint32_t it_bits = 0u;
  auto advance = [&]() -> bool {
    if (it_u >= 0 && it_sub + 1 < nsub) { it_sub++; return true; }
    while (it_bits == 0u) {
      if (++it_wi >= a.words) return false;
      it_bits = __builtin_amdgcn_readfirstlane(wgmask[it_wi]);
    }
    it_u = it_wi * 32 + __builtin_ctz(it_bits);
    it_bits &= it_bits - 1u;
    it_sub = 0;
    return true;
  };

  // ---- tile copies -------------------------------------------------------------
  const u32x4 k_rs = make_rsrc(a.k + b * a.ks_b + r * a.ks_h, (((int64_t)a.n_kv - 1) * a.ks_t + D) * 2);
  const u32x4 v_rs = make_rsrc(a.v + b * a.vs_b + r * a.vs_h, (((int64_t)a.n_kv - 1) * a.vs_t + D) * 2);
  const uint32_t lds0 = lds_addr_of(lds);
  const int c_row = (wave * 64 + lane) / C::NCH, c_pos = lane % C::NCH;
  const uint32_t k_off = (uint32_t)(c_row * (int)a.ks_t * 2 + ((c_pos ^ swz<D>(c_row)) << 4));
  const uint32_t v_off = (uint32_t)(c_row * (int)a.vs_t * 2 + ((c_pos ^ swz<D>(c_row)) << 4));
  const uint32_t k_step = (uint32_t)(C::ROWS_PER_COPY * (int)a.ks_t * 2);
  const uint32_t v_step = (uint32_t)(C::ROWS_PER_COPY * (int)a.vs_t * 2);

  // ---- operand read offsets ------------------------------------------------------
  // A operand: lane (n, h) reads logical chunk 2 ks + h of rows n, 32 + n.
  // Transposing read: lanes 16 g' .. 16 g' + 15 serve d columns 16 (g' & 1) .. + 15
  // of a d-tile and contraction half h = g' >> 1; lane s of the group points at
  // tile row 4 h + s / 4 (+ 8 for the second read), d offset 16 (g' & 1) + 4 (s % 4).
  const uint32_t a_rd = tile_off<D>(n, 8 * h);
  const int s16 = lane & 15, a16 = (lane >> 4) & 1;
  const uint32_t t_lo = tile_off<D>(4 * h + (s16 >> 2), 16 * a16 + 4 * (s16 & 3));
  const uint32_t t_hi = tile_off<D>(8 + 4 * h + (s16 >> 2), 16 * a16 + 4 * (s16 & 3));

  // first walk (GRAD = false): running max, sum of exponentials and sum of exponentials
  // times dP; D = <P, dP> = <dO, o> is taken from the latter two in fp32 (the stored bf16
  // output would put its rounding error into every dz of the row).  Second walk: both
  // come from the workspace.
  float m_run = -INFINITY, l_run = 0.f, dn_run = 0.f, lse2 = 0.f, dsum = 0.f;
  f32x16 dqacc[GRAD ? C::NDT : 1];
#pragma unroll
  for (int t = 0; t < (GRAD ? C::NDT : 1); t++) dqacc[t] = zero16();
  float db_acc = 0.f;
  if constexpr (GRAD) {
    const int64_t row = ((int64_t)b * a.h_q + my_head) * a.n_q + row_tok;
    lse2 = a.lse[row];
    dsum = a.dsum[row];
  }

  {
    constexpr bool grad = GRAD;
    float trk_next = (trk_ok && a.t_all > 0) ? trk_bias[0] : 0.f;
    float bias_row = 0.f;
    bool wave_on = false, diag = false;
    while (advance()) {
      const int cu = it_u, csub = it_sub;
      const uint32_t soff_k = (uint32_t)(cu * a.block + csub * 64) * (uint32_t)a.ks_t * 2u;
      const uint32_t soff_v = (uint32_t)(cu * a.block + csub * 64) * (uint32_t)a.vs_t * 2u;
      __syncthreads();                      // the previous tile is no longer read
#pragma unroll
      for (int c = 0; c < C::COPIES; c++) {
        copy16_to_lds(k_rs, lds0 + wave * 1024 + c * 4096, k_off, soff_k + c * k_step);
        copy16_to_lds(v_rs, lds0 + C::TILE_BYTES + wave * 1024 + c * 4096, v_off, soff_v + c * v_step);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();

      if (csub == 0) {
        wave_on = wave_ok && ((__builtin_amdgcn_readfirstlane(wvmask[wave * 64 + (cu >> 5)]) >> (cu & 31)) & 1u);
        diag = a.causal && cu == cw;
        if (wave_on) {
          float bt = 0.f;
          trk_has = false;
          if (!diag) {
            bt = -INFINITY;
            if (trk_ok) {
              if ((cu >> 5) != trk_wi) { trk_wi = cu >> 5; trk_word = trk_mask[trk_wi]; }
              if ((trk_word >> (cu & 31)) & 1u) {
                trk_has = true;
                bt = trk_next * kLog2e;
                if (grad) a.biasd[trk_base * a.t_all + cu] = trk_next;
                trk_rank++;
                if (trk_rank < a.t_all) trk_next = trk_bias[trk_rank];
              }
            }
          }
          bias_row = __shfl(bt, n / a.g_q);
        }
      }
      if (!wave_on) continue;
      const int kpos0 = cu * a.block + csub * 64;

      // the tile in two halves of 32 keys (keeps one S^T and one dP^T accumulator live)
      u32x4 pb[4];
      float dssum = 0.f;
      const float off = bias_row - lse2;
#pragma unroll
      for (int kt = 0; kt < 2; kt++) {
        // S^T = K Q^T, dP^T = V dO^T
        f32x16 s = zero16(), dp = zero16();
#pragma unroll
        for (int ks = 0; ks < D / 16; ks++) {
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_a<D>(k_t, a_rd, 2 * ks + kt), qf[ks], s, 0, 0, 0);
          if constexpr (GRAD)
            dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_a<D>(v_t, a_rd, 2 * ks + kt),
                                                         read_a<D>(do_t, do_rd, 2 * ks), dp, 0, 0, 0);
          else
            dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_a<D>(v_t, a_rd, 2 * ks + kt), dof[ks], dp, 0, 0, 0);
        }
        // key mask: causal inside the diagonal chunk, and the end of the sequence
        if (diag || kpos0 + 64 > a.n_kv) {
          const int k0 = kpos0 + 32 * kt + 4 * h;
          const int lim = min(diag ? row_pos - k0 : 0x7fffffff, a.n_kv - 1 - k0);
#pragma unroll
          for (int j = 0; j < 16; j++) {
            const int c = (j >> 2) * 8 + (j & 3);
            s[j] = c > lim ? -INFINITY : s[j];
          }
        }
        if (!grad) {
          float mloc = -INFINITY;
#pragma unroll
          for (int j = 0; j < 16; j++) mloc = fmaxf(mloc, s[j]);
          mloc = fmaxf(mloc, __shfl_xor(mloc, 32));
          const float tmax = fmaf(mloc, a.c1, bias_row);
          const float m_new = fmaxf(m_run, tmax);
          const float m_use = m_new == -INFINITY ? 0.f : m_new;
          float lsum = 0.f, dnsum = 0.f;
#pragma unroll
          for (int j = 0; j < 16; j++) {
            const float e = __builtin_amdgcn_exp2f(fmaf(s[j], a.c1, bias_row - m_use));
            lsum += e;
            dnsum = fmaf(e, dp[j], dnsum);
          }
          const float corr = __builtin_amdgcn_exp2f(m_run - m_use);
          l_run = l_run * corr + lsum;
          dn_run = dn_run * corr + dnsum;
          m_run = m_new;
        } else {
          // dS^T = P^T (dP^T - D), packed as the B operand of the second product
#pragma unroll
          for (int k = 0; k < 8; k++) {
            const int g = 2 * kt + (k >> 2), j = 8 * (k >> 2) + 2 * (k & 3);
            const float p0 = __builtin_amdgcn_exp2f(fmaf(s[j], a.c1, off));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(s[j + 1], a.c1, off));
            const float d0 = p0 * (dp[j] - dsum);
            const float d1 = p1 * (dp[j + 1] - dsum);
            dssum += d0 + d1;
            pb[g][k & 3] = cvt_bf16x2(d0, d1);
          }
        }
      }
      if constexpr (GRAD) {
      db_acc += dssum;
      // dQ^T += K^T dS^T
#pragma unroll
      for (int i = 0; i < C::NS; i++) {
        const int g = i / C::NDT, t = i % C::NDT;
        dqacc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_t<D>(k_t, t_lo, t_hi, g, t),
                                                           __builtin_bit_cast(bf16x8, pb[g]), dqacc[t], 0, 0, 0);
      }
      if (csub == nsub - 1) {
        // bias gradient of chunk cu: sum over the keys (both lane halves) and the
        // token's heads (adjacent lanes), written by the lane that tracks the token
        float tot = db_acc + __shfl_xor(db_acc, 32);
        for (int o = 1; o < a.g_q; o <<= 1) tot += __shfl_xor(tot, o);
        const float mine = __shfl(tot, (lane * a.g_q) & 31);
        if (!diag && trk_ok && trk_has) a.dbd[trk_base * a.t_all + cu] = mine;
        db_acc = 0.f;
      }
      }
    }
    if constexpr (!GRAD) {
      const float l_tot = l_run + __shfl_xor(l_run, 32);
      const float dn_tot = dn_run + __shfl_xor(dn_run, 32);
      lse2 = (m_run == -INFINITY ? 0.f : m_run) + __builtin_amdgcn_logf(l_tot);   // v_log_f32: log2
      dsum = l_tot > 0.f ? dn_tot / l_tot : 0.f;
    }
  }

  // ---- outputs -----------------------------------------------------------------
  if (row_ok) {
    const int64_t row = ((int64_t)b * a.h_q + my_head) * a.n_q + my_tok;
    if constexpr (!GRAD) {
      if (h == 0) { a.lse[row] = lse2; a.dsum[row] = dsum; }
    }
    float* dq = a.dq32 + row * D;
    if constexpr (GRAD)
#pragma unroll
    for (int t = 0; t < C::NDT; t++)
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
    const size_t nwords = (size_t)a.hb * a.t_all * a.cwords;
    hipLaunchKernelGGL(bwd_fill_zero_kernel, dim3((unsigned)((nwords + 255) / 256 < 1024 ? (nwords + 255) / 256 : 1024)),
                       dim3(256), 0, st, a.colmask, nwords);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  {
    const size_t lds = 2 * C::TILE_BYTES + 5 * 64 * 4;
    auto kern = bwd_q_kernel<D, false>;
    if ((e = allow_dyn_lds((const void*)kern, lds, done_lse)) != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(a.n_tiles * a.hb), dim3(256), lds, st, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  {
    const size_t lds = 4 * C::TILE_BYTES + 5 * 64 * 4;
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
