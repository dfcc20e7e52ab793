// Attention for fp32 tensors, forward (Stage 2 of Alg. 3 / Proposition 1 and the dense
// reference of Eq. 1) and backward, in fp32 throughout on the fp32 matrix cores
// (v_mfma_f32_16x16x4_f32: fp32 products, fp32 sums; 256 flop per clock and CU).
//
// Tiles and operand layouts: f32_tiles.h.
// A wave owns whole chunks (row kernels) or whole 16-row tiles (key kernel) and the waves of a
// workgroup add their results through LDS, so that the bias gradient of a chunk is one wave's and
// the launch is wide enough for a single head.
//
// What bounds it: at one head, 1024 tokens, d = 64, latency and launches (a wave has one chunk or
// two); at many heads the fp32 matrix rate.  Before (plain VALU kernels, dK / dV by one atomic
// per key and element): forward 138 us, backward rows 526 us, summary gradient 286 us on that shape.
#include <math.h>

#include "backward_args.h"
#include "common.h"
#include "dash_internal.h"
#include "f32_tiles.h"

namespace dash {

// e^(z - m) for logits in natural units: the difference is formed before the change of base, so a
// strong prior's large biases are rounded once, key by key, as in the logit itself.  The change of base is
// reduced first (Cody and Waite): 2^n 2^f with f = (z - m) log2(e) - n formed by two fused steps, log2(e) in two
// words.  v_exp_f32 of the product by one word instead rounds the argument: weights down to e^-20 of their row's
// largest were off by up to 9.6e-7, now by 1.1e-7, rms 3.6e-8, as with expf.  One head, 1024 tokens, forward and
// backward: 88.1 us with the one-word product, 91.2 now, 92.0 with expf and its range checks; correcting
// 2^(rounded product) by its residue afterwards takes 90.1 but rounds once more (rms 4.3e-8).  A difference below -200, -infinity among them, gives 0; NaN stays NaN (v_maximum3_f32).
constexpr float kLog2eLow = (float)(1.4426950408889634074 - (double)kLog2e);   // the second word
__device__ __forceinline__ float exp_diff(float z, float m) {
  const float t = __builtin_elementwise_maximum(z - m, -200.f);
  const float n = rintf(t * kLog2e);
  const float f = fmaf(t, kLog2eLow, fmaf(t, kLog2e, -n));
  return __builtin_ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
}

// The chunk list of a 16-row tile: union of its tokens' masks and, per token, the number of
// entries before each mask word (the bias lists are addressed by rank).
struct TileLists {
  uint32_t* uni;      // LDS [64]
  uint32_t* word;     // LDS [16][64]
  uint16_t* before;   // LDS [16][64]
  static constexpr size_t BYTES = 64 * 4 + 16 * 64 * 4 + 16 * 64 * 2;
  __device__ __forceinline__ TileLists(char* p)
      : uni((uint32_t*)p), word((uint32_t*)(p + 256)), before((uint16_t*)(p + 256 + 4096)) {}
  // mask: row of token 0 of the tile; ntok valid tokens.  Ends with a barrier.  All loads in flight together, and the ranks by DPP: one
  // token after the other, each load waited for, stood in front of every row kernel (one head, 1024 tokens, forward and backward: 83.0 -> 78 us with
  // the parts' records asked for in front of the lists and not one after the other; 16 heads x 2048 803 -> 784).
  template <int THREADS> __device__ __forceinline__ void build(const uint32_t* mask, int words, int ntok, int tid) {
    constexpr int NW = THREADS / 64, PER = 16 / NW;
    const int wave = tid >> 6, lane = tid & 63;
    uint32_t w[PER];
#pragma unroll
    for (int i = 0; i < PER; i++) {
      const int t = wave + i * NW;
      w[i] = t < ntok && lane < words ? mask[(int64_t)t * words + lane] : 0u;
    }
#pragma unroll
    for (int i = 0; i < PER; i++) {                   // rows of no token: empty
      const int t = wave + i * NW, mine = __popc(w[i]);
      word[t * 64 + lane] = w[i];
      before[t * 64 + lane] = (uint16_t)(wave_scan(mine) - mine);
    }
    __syncthreads();
    if (tid < 64) {
      uint32_t u = 0u;
#pragma unroll
      for (int t = 0; t < 16; t++) u |= word[t * 64 + tid];
      uni[tid] = u;
    }
    __syncthreads();
  }
  __device__ __forceinline__ bool has(int t, int c) const { return (word[t * 64 + (c >> 5)] >> (c & 31)) & 1u; }
  __device__ __forceinline__ int rank(int t, int c) const {
    return before[t * 64 + (c >> 5)] + __popc(word[t * 64 + (c >> 5)] & ((1u << (c & 31)) - 1u));
  }
};

// Walks the set bits of the union that belong to worker `who` of `of` (every of-th entry).
struct ListWalk {
  const uint32_t* uni;
  int words, wi, skip, of;
  uint32_t bits;
  __device__ __forceinline__ ListWalk(const uint32_t* u, int words_, int who, int of_)
      : uni(u), words(words_), wi(-1), skip(who), of(of_), bits(0u) {}
  __device__ __forceinline__ int next() {     // chunk id, or -1 (wave-uniform)
    for (;;) {
      while (bits == 0u) {
        if (++wi >= words) return -1;
        bits = __builtin_amdgcn_readfirstlane(uni[wi]);
      }
      const int c = wi * 32 + __builtin_ctz(bits);
      bits &= bits - 1u;
      if (skip-- == 0) { skip = of - 1; return c; }
    }
  }
};

// ---------------------------------------------------------------------------
// Forward
// ---------------------------------------------------------------------------
struct S2FArgs {
  const float* q; const float* k; const float* v; float* o;
  const uint32_t* mask; const float* bias;
  int h_kv, g_q, n_q, n_kv, block, t_all, words, pos0, causal, hb, n_tiles;
  int64_t qs_b, qs_h, qs_t, ks_b, ks_h, ks_t, vs_b, vs_h, vs_t, os_b, os_h, os_t;
  float scale;
};

template <int D, bool DENSE>
__global__ __launch_bounds__(512) void s2_f32_kernel(S2FArgs a) {
  using C = F32Cfg<D>;
  constexpr int NWV = 8;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  float* tiles = reinterpret_cast<float*>(lds);                       // [8][16][LD]
  float* ms = tiles + NWV * 16 * C::LD;                               // [8][16]
  float* ls = ms + NWV * 16;                                          // [8][16]
  TileLists tl(reinterpret_cast<char*>(ls + NWV * 16));
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, hq = lane >> 4;
  const int hbi = blockIdx.x % a.hb, tile = a.n_tiles - 1 - blockIdx.x / a.hb;   // longest rows first
  const int r = hbi % a.h_kv, b = hbi / a.h_kv;
  const int tokt = 16 / a.g_q, tok0 = tile * tokt, ntok = min(tokt, a.n_q - tok0);
  const int t_n = min(n / a.g_q, ntok - 1), tok = tok0 + t_n;          // this lane's row (padding repeats the last token)
  const int pos = a.pos0 + tok, cw = (a.pos0 + tok0) / a.block;       // all tokens of a tile lie in one chunk
  const int nsub = a.block >> 4;
  const int64_t base = ((int64_t)b * a.h_kv + r) * a.n_q + tok0;
  if (DENSE) {
    if (tid < 64) {
      const int last = a.causal ? cw : a.t_all - 1, lo = tid * 32;
      tl.uni[tid] = last < lo ? 0u : (last - lo >= 31 ? 0xffffffffu : (2u << (last - lo)) - 1u);
    }
    __syncthreads();
  } else {
    tl.build<512>(a.mask + base * a.words, a.words, ntok, tid);
  }
  f32x4 qf[C::NS];
  load_row<D>(a.q + b * a.qs_b + (int64_t)(r * a.g_q + n % a.g_q) * a.qs_h + (int64_t)tok * a.qs_t, hq, qf);
  const float* kb = a.k + b * a.ks_b + r * a.ks_h;
  const float* vb = a.v + b * a.vs_b + r * a.vs_h;
  float m_run = -INFINITY, l_run = 0.f;       // l_run: this lane's keys only
  f32x4 o[C::NS];
#pragma unroll
  for (int i = 0; i < C::NS; i++) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  ListWalk it(tl.uni, DENSE ? 64 : a.words, wave, NWV);
  for (int c = it.next(); c >= 0; c = it.next()) {
    const bool diag = a.causal && c == cw;
    const bool mine = DENSE || tl.has(t_n, c);
    float bias = 0.f;
    if (!DENSE && !diag && mine) bias = a.bias[(base + t_n) * a.t_all + tl.rank(t_n, c)];
    // SUB sub-tiles of 16 keys per step: all K loads of a step are in flight together, and its V loads
    // are issued before the softmax that they wait behind
    constexpr int SUB = D == 64 ? 4 : 2;
    for (int st0 = 0; st0 < nsub; st0 += SUB) {
      const int kpos0 = c * a.block + st0 * 16;
      if (kpos0 >= a.n_kv || (diag && kpos0 > a.pos0 + tok0 + ntok - 1)) break;
      f32x4 kf[SUB][C::NS], vr[SUB][4][C::NV], s[SUB];
#pragma unroll
      for (int st = 0; st < SUB; st++) load_row<D>(kb + (int64_t)min(kpos0 + 16 * st + n, a.n_kv - 1) * a.ks_t, hq, kf[st]);
#pragma unroll
      for (int st = 0; st < SUB; st++)
#pragma unroll
        for (int t = 0; t < 4; t++) load_row2<D>(vb + (int64_t)min(kpos0 + 16 * st + 4 * hq + t, a.n_kv - 1) * a.vs_t, n, vr[st][t]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int st = 0; st < SUB; st++) s[st] = mma_dot<D>(kf[st], qf);
      // dead keys: after the row's position, past the end of the sequence, of a chunk the row did not keep
      const int lim = mine ? min(diag ? pos : 0x7fffffff, a.n_kv - 1) - kpos0 - 4 * hq : -1;
      float mx = -INFINITY;
#pragma unroll
      for (int st = 0; st < SUB; st++)
#pragma unroll
        for (int v = 0; v < 4; v++) {
          s[st][v] = 16 * st + v > lim ? -INFINITY : fmaf(s[st][v], a.scale, bias);
          mx = fmaxf(mx, s[st][v]);
        }
      const float m_new = fmaxf(m_run, quad_rows_max(mx));
      const float m_use = m_new == -INFINITY ? 0.f : m_new;
      const float corr = exp_diff(m_run, m_use);
      m_run = m_new;
      l_run *= corr;
#pragma unroll
      for (int i = 0; i < C::NS; i++) o[i] *= corr;
#pragma unroll
      for (int st = 0; st < SUB; st++) {
#pragma unroll
        for (int t = 0; t < 4; t++) s[st][t] = exp_diff(s[st][t], m_use);
        l_run += (s[st][0] + s[st][1]) + (s[st][2] + s[st][3]);
      }
      mma_outer_keys<D, SUB>(vr, s, lim, ntok, a.g_q, lane, o);
    }
  }
  // ---- add up the waves: rows weighted by e^(m_wave - M) --------------------------------------
  const float l_tot = quad_rows_sum(l_run);
  if (hq == 0) { ms[wave * 16 + n] = m_run; ls[wave * 16 + n] = l_tot; }
  __syncthreads();
  float M = -INFINITY, den = 0.f;
#pragma unroll
  for (int w = 0; w < NWV; w++) M = fmaxf(M, ms[w * 16 + n]);
#pragma unroll
  for (int w = 0; w < NWV; w++) den = fmaf(ms[w * 16 + n] == -INFINITY ? 0.f : exp_diff(ms[w * 16 + n], M), ls[w * 16 + n], den);
  put_tile<D>(tiles + wave * 16 * C::LD, n, hq, o, m_run == -INFINITY ? 0.f : exp_diff(m_run, M) / den);
  __syncthreads();
  for (int i = tid; i < 16 * D / 4; i += 512) {
    const int row = i / (D / 4), d4 = (i % (D / 4)) * 4;
    if (row / a.g_q >= ntok) continue;
    f32x4 x = *reinterpret_cast<const f32x4*>(tiles + row * C::LD + d4);
#pragma unroll
    for (int w = 1; w < NWV; w++) x += *reinterpret_cast<const f32x4*>(tiles + (w * 16 + row) * C::LD + d4);
    *reinterpret_cast<f32x4*>(a.o + b * a.os_b + (int64_t)(r * a.g_q + row % a.g_q) * a.os_h +
                              (int64_t)(tok0 + row / a.g_q) * a.os_t + d4) = x;
  }
}

template <int D, bool DENSE> static hipError_t launch_s2_f32_t(const S2FArgs& a, hipStream_t st) {
  constexpr size_t lds = (size_t)(8 * 16 * F32Cfg<D>::LD + 2 * 8 * 16) * 4 + TileLists::BYTES;
  auto kern = s2_f32_kernel<D, DENSE>;
  static LdsOptIn opt_in;
  if (hipError_t e = allow_dyn_lds((const void*)kern, lds, opt_in); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(a.n_tiles * a.hb)), dim3(512), lds, st, a);
  return hipGetLastError();
}

hipError_t launch_s2_f32(const dash_params& p, const Layout& L, const void* q, const void* k,
                         const void* v, void* o, const uint32_t* mask, const float* bias,
                         bool dense, hipStream_t st) {
  S2FArgs a;
  a.q = (const float*)q; a.k = (const float*)k; a.v = (const float*)v; a.o = (float*)o;
  a.mask = mask; a.bias = bias;
  a.h_kv = p.h_kv; a.g_q = L.g_q; a.n_q = p.n_q; a.n_kv = p.n_kv; a.block = p.block_size;
  a.t_all = L.t_all; a.words = L.words; a.pos0 = L.pos0; a.causal = p.causal;
  a.hb = p.h_kv * p.batch;
  const int tokt = 16 / L.g_q;
  a.n_tiles = (p.n_q + tokt - 1) / tokt;
  a.qs_b = p.q_stride[0]; a.qs_h = p.q_stride[1]; a.qs_t = p.q_stride[2];
  a.ks_b = p.k_stride[0]; a.ks_h = p.k_stride[1]; a.ks_t = p.k_stride[2];
  a.vs_b = p.v_stride[0]; a.vs_h = p.v_stride[1]; a.vs_t = p.v_stride[2];
  a.os_b = p.o_stride[0]; a.os_h = p.o_stride[1]; a.os_t = p.o_stride[2];
  a.scale = L.scale;
  if (p.head_dim == 128) return dense ? launch_s2_f32_t<128, true>(a, st) : launch_s2_f32_t<128, false>(a, st);
  return dense ? launch_s2_f32_t<64, true>(a, st) : launch_s2_f32_t<64, false>(a, st);
}

// ---------------------------------------------------------------------------
// Backward (n_q == n_kv; see backward.hip for the chain)
// ---------------------------------------------------------------------------
// Row kernel, one workgroup of 4 waves per (16-row tile, part of its chunk list).
//   GRAD = false: log-sum-exp and D per row, or, of several parts, (max, sum, sum of exponentials
//     times dP) of the part's keys into `scratch`; also clears what the later kernels add to (dq32, and dk, dv, dkbar if `clear_kv`).
//   GRAD = true: log-sum-exp and D (from the parts' records); bias gradient and a copy of the bias
//     by chunk id; dq (attention part) added to dq32.
struct RowF32 {
  int parts, n_tiles, clear_kv;
  int64_t rows;         // batch * h_q * n_q
  float* scratch;       // parts > 1: [parts][rows][3]
};

template <int D, bool GRAD>
__global__ __launch_bounds__(256, 2) void bwd_f32_row_kernel(BwdArgs a, RowF32 x) {
  using C = F32Cfg<D>;
  constexpr int NWV = 4;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  TileLists tl(lds);
  float* red = reinterpret_cast<float*>(lds + TileLists::BYTES);      // GRAD: [4][16][LD]; else [4][16][3]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, hq = lane >> 4;
  const int hbi = blockIdx.x % a.hb, tile = x.n_tiles - 1 - blockIdx.x / a.hb, part = blockIdx.y;
  const int r = hbi % a.h_kv, b = hbi / a.h_kv;
  const int tokt = 16 / a.g_q, tok0 = tile * tokt, ntok = min(tokt, a.n_q - tok0);
  const int t_n = min(n / a.g_q, ntok - 1), tok = tok0 + t_n, head = r * a.g_q + n % a.g_q;
  const int cw = tok0 / a.block, nsub = a.block >> 4;
  const int64_t base = ((int64_t)b * a.h_kv + r) * a.n_q + tok0;
  const bool row_ok = n / a.g_q < ntok;
  const int64_t row_n = ((int64_t)b * a.h_q + head) * a.n_q + tok;
  if (!GRAD) {
    const int64_t step = (int64_t)gridDim.x * gridDim.y * 256, i0 = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * 256 + tid;
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    const int64_t nq4 = (int64_t)a.hb * a.g_q * a.n_q * (D / 4);
    for (int64_t i = i0; i < nq4; i += step) reinterpret_cast<f32x4*>(a.dq32)[i] = z;
    if (x.clear_kv) {
      const int64_t nk4 = (int64_t)a.hb * a.n_kv * (D / 4);
      for (int64_t i = i0; i < nk4; i += step) {
        const int64_t row = i / (D / 4);
        const int key = (int)(row % a.n_kv), e = (int)(i % (D / 4)) * 4;
        const int64_t bb = row / a.n_kv / a.h_kv, rr = row / a.n_kv % a.h_kv;
        *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.dk) + bb * a.ks_b + rr * a.ks_h + (int64_t)key * a.ks_t + e) = z;
        *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.dv) + bb * a.vs_b + rr * a.vs_h + (int64_t)key * a.vs_t + e) = z;
      }
      if (a.dkbar_out) {
        const int64_t nb4 = (int64_t)a.hb * a.t_c * (D / 4);
        for (int64_t i = i0; i < nb4; i += step) reinterpret_cast<f32x4*>(a.dkbar_out)[i] = z;
      }
    }
  }
  f32x4 qf[C::NS], of[C::NS];
  load_row<D>(reinterpret_cast<const float*>(a.q) + b * a.qs_b + head * a.qs_h + (int64_t)tok * a.qs_t, hq, qf);
  load_row<D>(reinterpret_cast<const float*>(a.d_o) + b * a.os_b + head * a.os_h + (int64_t)tok * a.os_t, hq, of);
  // GRAD: the parts' records (max, sum, sum times dP), four at a time; the first four arrive with the lists
  float rec[4][3];
  auto ask_parts = [&](int p0) {
    const float* rp = x.scratch + row_n * 3;
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
      for (int e = 0; e < 3; e++) rec[i][e] = rp[min(p0 + i, x.parts - 1) * x.rows * 3 + e];
  };
  if constexpr (GRAD) { if (x.parts > 1) ask_parts(0); }
  tl.build<256>(a.mask + base * a.words, a.words, ntok, tid);
  const float* kb = reinterpret_cast<const float*>(a.k) + b * a.ks_b + r * a.ks_h;
  const float* vb = reinterpret_cast<const float*>(a.v) + b * a.vs_b + r * a.vs_h;
  float m_run = -INFINITY, l_run = 0.f, dn_run = 0.f;     // of this lane's keys
  float lse = 0.f, dsum = 0.f;
  f32x4 dq[GRAD ? C::NS : 1];
  if constexpr (GRAD) {
#pragma unroll
    for (int i = 0; i < C::NS; i++) dq[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (x.parts == 1) {
      lse = a.lse[row_n];
      dsum = a.dsum[row_n];
    } else {
      float M = -INFINITY, l = 0.f, dn = 0.f;
      for (int p0 = 0; p0 < x.parts; p0 += 4) {
        if (p0 > 0) ask_parts(p0);
        float m_new = M;
#pragma unroll
        for (int i = 0; i < 4; i++) m_new = fmaxf(m_new, rec[i][0]);
        const float f = M == -INFINITY ? 0.f : exp_diff(M, m_new);
        l *= f;
        dn *= f;
        M = m_new;
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const float w = rec[i][0] == -INFINITY || p0 + i >= x.parts ? 0.f : exp_diff(rec[i][0], M);
          l = fmaf(w, rec[i][1], l);
          dn = fmaf(w, rec[i][2], dn);
        }
      }
      lse = M + logf(l);
      dsum = dn / l;
      if (part == 0 && wave == 0 && hq == 0 && row_ok) { a.lse[row_n] = lse; a.dsum[row_n] = dsum; }
    }
  }
  ListWalk it(tl.uni, a.words, part * NWV + wave, x.parts * NWV);
  for (int c = it.next(); c >= 0; c = it.next()) {
    const bool diag = a.causal && c == cw, mine = tl.has(t_n, c);
    float bias = 0.f, db = 0.f;
    if (!diag && mine) bias = a.bias[(base + t_n) * a.t_all + tl.rank(t_n, c)];
    // SUB sub-tiles of 16 keys per round trip; more of them cost waves (at four, 190 registers: 16 heads x 2047 tokens 962 -> 997 us)
    constexpr int SUB = D == 64 && !GRAD ? 2 : 1;
    for (int st0 = 0; st0 < nsub; st0 += SUB) {
      const int kpos0 = c * a.block + st0 * 16;
      if (kpos0 >= a.n_kv || (diag && kpos0 > tok0 + ntok - 1)) break;
      f32x4 kf[SUB][C::NS], vf[SUB][C::NS], kr[SUB][4][C::NV], s[SUB], dp[SUB];
#pragma unroll
      for (int st = 0; st < SUB; st++) {
        load_row<D>(kb + (int64_t)min(kpos0 + 16 * st + n, a.n_kv - 1) * a.ks_t, hq, kf[st]);
        load_row<D>(vb + (int64_t)min(kpos0 + 16 * st + n, a.n_kv - 1) * a.vs_t, hq, vf[st]);
      }
      if constexpr (GRAD) {
#pragma unroll
        for (int st = 0; st < SUB; st++)
#pragma unroll
          for (int t = 0; t < 4; t++) load_row2<D>(kb + (int64_t)min(kpos0 + 16 * st + 4 * hq + t, a.n_kv - 1) * a.ks_t, n, kr[st][t]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int st = 0; st < SUB; st++) { s[st] = mma_dot<D>(kf[st], qf); dp[st] = mma_dot<D>(vf[st], of); }
      const int lim = mine ? min(diag ? tok : 0x7fffffff, a.n_kv - 1) - kpos0 - 4 * hq : -1;   // as in the forward
      if constexpr (!GRAD) {
        float mx = m_run;
#pragma unroll
        for (int st = 0; st < SUB; st++)
#pragma unroll
          for (int v = 0; v < 4; v++) {
            s[st][v] = 16 * st + v > lim ? -INFINITY : fmaf(s[st][v], a.scale, bias);
            mx = fmaxf(mx, s[st][v]);
          }
        const float m_use = mx == -INFINITY ? 0.f : mx;
        const float corr = exp_diff(m_run, m_use);
        m_run = mx;
        float dn = 0.f, l = 0.f;
#pragma unroll
        for (int st = 0; st < SUB; st++) {
#pragma unroll
          for (int v = 0; v < 4; v++) {
            s[st][v] = exp_diff(s[st][v], m_use);
            dn = fmaf(s[st][v], 16 * st + v > lim ? 0.f : dp[st][v], dn);
          }
          l += (s[st][0] + s[st][1]) + (s[st][2] + s[st][3]);
        }
        l_run = fmaf(l_run, corr, l);
        dn_run = fmaf(dn_run, corr, dn);
      } else {
#pragma unroll
        for (int st = 0; st < SUB; st++)
#pragma unroll
          for (int t = 0; t < 4; t++) {
            s[st][t] = 16 * st + t > lim ? 0.f : exp_diff(fmaf(s[st][t], a.scale, bias), lse) * (dp[st][t] - dsum);
            db += s[st][t];
          }
        mma_outer_keys<D, SUB>(kr, s, lim, ntok, a.g_q, lane, dq);
      }
    }
    if constexpr (GRAD) {
      // bias gradient: over the chunk's keys (four lanes of the row) and the group's heads (rows)
      db = quad_rows_sum(db);
      for (int o = 1; o < a.g_q; o <<= 1) db += __shfl_xor(db, o);
      if (!diag && mine && row_ok && hq == 0 && n % a.g_q == 0) {
        a.dbd[(base + t_n) * a.t_all + c] = db;
        a.biasd[(base + t_n) * a.t_all + c] = bias;
      }
    }
  }
  if constexpr (!GRAD) {
    const float M = quad_rows_max(m_run), w = m_run == -INFINITY ? 0.f : exp_diff(m_run, M);
    const float l = quad_rows_sum(l_run * w), dn = quad_rows_sum(dn_run * w);
    if (hq == 0) { red[(wave * 16 + n) * 3] = M; red[(wave * 16 + n) * 3 + 1] = l; red[(wave * 16 + n) * 3 + 2] = dn; }
    __syncthreads();
    if (tid < 16) {
      float Mt = -INFINITY, lt = 0.f, dt = 0.f;
      for (int w_ = 0; w_ < NWV; w_++) Mt = fmaxf(Mt, red[(w_ * 16 + tid) * 3]);
      for (int w_ = 0; w_ < NWV; w_++) {
        const float e = red[(w_ * 16 + tid) * 3] == -INFINITY ? 0.f : exp_diff(red[(w_ * 16 + tid) * 3], Mt);
        lt = fmaf(e, red[(w_ * 16 + tid) * 3 + 1], lt);
        dt = fmaf(e, red[(w_ * 16 + tid) * 3 + 2], dt);
      }
      if (row_ok) {     // wave 0, lane tid: row_n is row tid
        if (x.parts == 1) {
          a.lse[row_n] = Mt + logf(lt);
          a.dsum[row_n] = dt / lt;
        } else {
          float* rp = x.scratch + (part * x.rows + row_n) * 3;
          rp[0] = Mt; rp[1] = lt; rp[2] = dt;
        }
      }
    }
  } else {
    put_tile<D>(red + wave * 16 * C::LD, n, hq, dq, a.scale);
    __syncthreads();
    for (int i = tid; i < 16 * D; i += 256) {
      const int row = i / D, d = i % D;
      if (row / a.g_q >= ntok) continue;
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < NWV; w++) v += red[(w * 16 + row) * C::LD + d];
      float* dst = a.dq32 + (((int64_t)b * a.h_q + r * a.g_q + row % a.g_q) * a.n_q + tok0 + row / a.g_q) * D + d;
      if (x.parts == 1) *dst = v; else unsafeAtomicAdd(dst, v);
    }
  }
}

// Key kernel, one workgroup of 4 waves per (16-key tile, part of the rows that attend its chunk):
// dK, dV and the chunk's summary gradient.  Several parts add to cleared outputs.
// At d = 64 the bound keeps two waves per SIMD: without it 196 + 64 registers, four more than allow that, and the 512
// workgroups of a small launch ran in two rounds.  With it 218, and the per-row values asked for before the rows: one
// head, 1024 tokens 23 -> 15 us; backward pass of 16 heads x 2048 tokens 765 -> 577 us, of 8 / 4 heads x 3000 in chunks
// of 128 839 -> 626.  At d = 128 (one wave) 4 heads over one, 1500 tokens: 343 -> 312.
template <int D>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void bwd_f32_key_kernel(BwdArgs a, int parts) {
  using C = F32Cfg<D>;
  constexpr int NWV = 4;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  float* red = reinterpret_cast<float*>(lds);                         // [4][16][LD]
  float* kbs = red + NWV * 16 * C::LD;                                // [4][D]
  uint32_t* bits = reinterpret_cast<uint32_t*>(kbs + NWV * D);        // [n_q / 32]: tokens that attend the chunk
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, hq = lane >> 4;
  const int hbi = blockIdx.x % a.hb, ktile = blockIdx.x / a.hb, part = blockIdx.y;   // early keys (the most rows) first
  const int r = hbi % a.h_kv, b = hbi / a.h_kv;
  const int kpos0 = ktile * 16, c = kpos0 / a.block;
  const int tokt = 16 / a.g_q;
  const int64_t mrow = ((int64_t)b * a.h_kv + r) * a.n_q;
  // the tokens of this part: whole 64-token groups, dealt out evenly over those that can attend the keys
  const int g0 = a.causal ? kpos0 / 64 : 0, ng = (a.n_q + 63) / 64 - g0;
  const int per = (ng + parts - 1) / parts;
  const int gb = g0 + part * per, ge = min(gb + per, g0 + ng);
  for (int g = gb + wave; g < ge; g += NWV) {
    const int tk = g * 64 + lane;
    const bool bit = tk < a.n_q && ((a.mask[(mrow + tk) * a.words + (c >> 5)] >> (c & 31)) & 1u);
    const uint64_t bal = __ballot(bit);
    if (lane == 0) { bits[2 * (g - gb)] = (uint32_t)bal; bits[2 * (g - gb) + 1] = (uint32_t)(bal >> 32); }
  }
  const int key = min(kpos0 + n, a.n_kv - 1);
  f32x4 kf[C::NS], vf[C::NS];
  load_row<D>(reinterpret_cast<const float*>(a.k) + b * a.ks_b + r * a.ks_h + (int64_t)key * a.ks_t, hq, kf);
  load_row<D>(reinterpret_cast<const float*>(a.v) + b * a.vs_b + r * a.vs_h + (int64_t)key * a.vs_t, hq, vf);
  __syncthreads();
  const float* qb = reinterpret_cast<const float*>(a.q) + b * a.qs_b + (int64_t)r * a.g_q * a.qs_h;
  const float* ob = reinterpret_cast<const float*>(a.d_o) + b * a.os_b + (int64_t)r * a.g_q * a.os_h;
  f32x4 dk[C::NS], dv[C::NS], kbar[C::NV];
#pragma unroll
  for (int i = 0; i < C::NS; i++) { dk[i] = f32x4{0.f, 0.f, 0.f, 0.f}; dv[i] = dk[i]; }
#pragma unroll
  for (int i = 0; i < C::NV; i++) kbar[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int tpg = 64 / tokt;                  // row tiles per 64-token group
  for (int T = gb * tpg + wave; T < ge * tpg; T += NWV) {
    const int tok0 = T * tokt;
    if (tok0 >= a.n_q) break;
    const int lt = tok0 - gb * 64;
    const uint32_t tb = (__builtin_amdgcn_readfirstlane(bits[lt >> 5]) >> (lt & 31)) & (tokt == 32 ? ~0u : (1u << tokt) - 1u);
    if (tb == 0u) continue;                   // bits of tokens past the end are 0
    // per-row values: lane (m, kq) fetches one of the four of row m, then every lane takes its rows'
    const int cdiag = tok0 / a.block;
    const bool isdiag = a.causal && c == cdiag;
    const int n_cand = a.causal ? max(cdiag - a.window, 0) : a.t_c;
    float val;
    bool val_ok = true;                       // else not written
    {
      const int tk = min(tok0 + n / a.g_q, a.n_q - 1);
      const int64_t hrow = ((int64_t)b * a.h_q + r * a.g_q + n % a.g_q) * a.n_q + tk;
      const bool bit = (tb >> (n / a.g_q)) & 1u;
      if (hq >= 2) val_ok = bit && (hq == 2 ? !isdiag : c < n_cand);
      const float* vp = hq == 0 ? a.lse + hrow : hq == 1 ? a.dsum + hrow : hq == 2 ? a.biasd + (mrow + tk) * a.t_all + c : a.dxd + hrow * a.t_all + c;
      val = *vp;
    }
    // all loads of the row tile in flight together
    const int64_t ra = min(tok0 + n / a.g_q, a.n_q - 1);
    f32x4 qa[C::NS], oa[C::NS], qw[1][4][C::NV], ow[1][4][C::NV];
    load_row<D>(qb + (n % a.g_q) * a.qs_h + ra * a.qs_t, hq, qa);
    load_row<D>(ob + (n % a.g_q) * a.os_h + ra * a.os_t, hq, oa);
#pragma unroll
    for (int t = 0; t < 4; t++) {
      const int row = 4 * hq + t;
      const int64_t rt = min(tok0 + row / a.g_q, a.n_q - 1);
      load_row2<D>(ob + (row % a.g_q) * a.os_h + rt * a.os_t, n, ow[0][t]);
      load_row2<D>(qb + (row % a.g_q) * a.qs_h + rt * a.qs_t, n, qw[0][t]);
    }
    val = val_ok ? val : 0.f;
    float bs[4], ls[4], ds[4], dx[4];
#pragma unroll
    for (int v = 0; v < 4; v++) {
      const int row = 4 * hq + v;
      ls[v] = __shfl(val, row);
      bs[v] = __shfl(val, 32 + row);
      ds[v] = __shfl(val, 16 + row);
      dx[v] = __shfl(val, 48 + row);
    }
    const f32x4 s = mma_dot<D>(qa, kf), dp = mma_dot<D>(oa, vf);
    // tokens of the tile that do not attend this lane's key: the chunk not kept, or the key after them
    uint32_t dead = ~tb & ((1u << tokt) - 1u);
    if (a.causal && kpos0 + n > tok0) dead |= (1u << min(kpos0 + n - tok0, tokt)) - 1u;
    f32x4 p, dz;
#pragma unroll
    for (int t = 0; t < 4; t++) {
      const bool off = (dead >> ((4 * hq + t) / a.g_q)) & 1u;
      p[t] = off ? 0.f : exp_diff(fmaf(s[t], a.scale, bs[t]), ls[t]);
      dz[t] = off ? 0.f : p[t] * (dp[t] - ds[t]);
    }
    mma_outer_rows<D>(ow, p, dead, a.g_q, lane, dv);
    mma_outer_rows<D>(qw, dz, dead, a.g_q, lane, dk);
#pragma unroll
    for (int t = 0; t < 4; t++)
#pragma unroll
      for (int nv = 0; nv < C::NV; nv++)
#pragma unroll
        for (int e = 0; e < 4; e++) kbar[nv][e] = dx[t] == 0.f ? kbar[nv][e] : fmaf(qw[0][t][nv][e], dx[t], kbar[nv][e]);
  }
  // ---- add up the waves ------------------------------------------------------------------------
#pragma unroll
  for (int nv = 0; nv < C::NV; nv++)
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const float t = quad_rows_sum(kbar[nv][e]);
      if (hq == 0) kbs[wave * D + 64 * nv + 4 * n + e] = t;
    }
  put_tile<D>(red + wave * 16 * C::LD, n, hq, dk, a.scale);
  __syncthreads();
  const bool fold = c < a.t_c && !a.dkbar_out;
  const float kscale = a.xscale / (float)a.block;
  for (int i = tid; i < 16 * D; i += 256) {
    const int row = i / D, d = i % D;
    if (kpos0 + row >= a.n_kv) continue;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < NWV; w++) v += red[(w * 16 + row) * C::LD + d];
    // block-mean summaries: every key of a complete chunk receives 1/B of the chunk's dkbar
    if (fold) v = fmaf((kbs[d] + kbs[D + d]) + (kbs[2 * D + d] + kbs[3 * D + d]), kscale, v);
    float* dst = reinterpret_cast<float*>(a.dk) + b * a.ks_b + r * a.ks_h + (int64_t)(kpos0 + row) * a.ks_t + d;
    if (parts == 1) *dst = v; else unsafeAtomicAdd(dst, v);
  }
  if (a.dkbar_out && c < a.t_c && kpos0 % a.block == 0) {
    for (int d = tid; d < D; d += 256) {
      const float v = ((kbs[d] + kbs[D + d]) + (kbs[2 * D + d] + kbs[3 * D + d])) * a.xscale;
      float* dst = a.dkbar_out + (((int64_t)b * a.h_kv + r) * a.t_c + c) * D + d;
      if (parts == 1) *dst = v; else unsafeAtomicAdd(dst, v);
    }
  }
  __syncthreads();
  put_tile<D>(red + wave * 16 * C::LD, n, hq, dv, 1.f);
  __syncthreads();
  for (int i = tid; i < 16 * D; i += 256) {
    const int row = i / D, d = i % D;
    if (kpos0 + row >= a.n_kv) continue;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < NWV; w++) v += red[(w * 16 + row) * C::LD + d];
    float* dst = reinterpret_cast<float*>(a.dv) + b * a.vs_b + r * a.vs_h + (int64_t)(kpos0 + row) * a.vs_t + d;
    if (parts == 1) *dst = v; else unsafeAtomicAdd(dst, v);
  }
}

static int clamp_int(int64_t x, int lo, int hi) { return x < lo ? lo : (x > hi ? hi : (int)x); }

// Parts: enough workgroups for two per CU, while a wave keeps at least one chunk (rows) or a
// part one 64-token group (keys).  The rows' records fit the score-gradient array they
// are kept in until the routing kernel fills it: 3 floats per row and part of its t_all >= 4 parts.
static int key_parts(const BwdArgs& a) {
  const int ktiles = (a.n_kv + 15) / 16;
  return clamp_int(512 / ((int64_t)ktiles * a.hb), 1, (a.n_q + 63) / 64);
}

template <int D> static hipError_t launch_rows_t(const BwdArgs& a, hipStream_t st) {
  RowF32 x;
  const int tokt = 16 / a.g_q;
  x.n_tiles = (a.n_q + tokt - 1) / tokt;
  x.parts = clamp_int(512 / ((int64_t)x.n_tiles * a.hb), 1, a.t_all >= 4 ? a.t_all / 4 : 1);
  x.rows = (int64_t)a.hb * a.g_q * a.n_q;
  x.clear_kv = key_parts(a) > 1;
  x.scratch = a.dxd;
  const dim3 grid((unsigned)(x.n_tiles * a.hb), (unsigned)x.parts), blk(256);
  hipLaunchKernelGGL((bwd_f32_row_kernel<D, false>), grid, blk, TileLists::BYTES + 4 * 16 * 3 * 4, st, a, x);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  hipLaunchKernelGGL((bwd_f32_row_kernel<D, true>), grid, blk, TileLists::BYTES + 4 * 16 * F32Cfg<D>::LD * 4, st, a, x);
  return hipGetLastError();
}

template <int D> static hipError_t launch_keys_t(const BwdArgs& a, hipStream_t st) {
  const int parts = key_parts(a), ktiles = (a.n_kv + 15) / 16;
  const size_t lds = (size_t)(4 * 16 * F32Cfg<D>::LD + 4 * D) * 4 + (size_t)((a.n_q + 63) / 64) * 8;
  auto kern = bwd_f32_key_kernel<D>;
  static LdsOptIn opt_in;
  if (hipError_t e = allow_dyn_lds((const void*)kern, lds, opt_in); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(ktiles * a.hb), (unsigned)parts), dim3(256), lds, st, a, parts);
  return hipGetLastError();
}

hipError_t launch_bwd_f32_rows(const BwdArgs& a, int head_dim, hipStream_t st) {
  return head_dim == 128 ? launch_rows_t<128>(a, st) : launch_rows_t<64>(a, st);
}
hipError_t launch_bwd_f32_keys(const BwdArgs& a, int head_dim, hipStream_t st) {
  return head_dim == 128 ? launch_keys_t<128>(a, st) : launch_keys_t<64>(a, st);
}

}  // namespace dash
