// The decode kernel: one query token per sequence attends its routed chunks with the Stage-1
// bias added to the logits (Sec. 3.3 Eq. 6 in the bias form of Proposition 1; Alg. 3), the
// attended list cut into splits whose partial results are merged (Sec. 3.5).  One template:
//   DEC_ROUTE  the whole step in one launch: scores, entmax threshold, list, attention, merge
//   DEC_LISTS  attention over lists read from memory (dash_stage2_attend)
//   DEC_DENSE  the dense reference (Eq. 1)
//
// The step is bound by HBM: every attended chunk is read once (K and V rows, 2 * block * d * 2
// bytes) and used for 4 * g_q flops per byte, plus the summaries of the candidates.  Short caches
// are bound by latency instead: launches and dependent round trips to memory.
//
// Attention.  A workgroup (4 waves) owns the 32-key sub-tiles [t0, t1) of one (batch, kv-head)
// pair's ascending list and streams them global -> LDS (buffer_load ... lds, no staging
// registers): NST - 1 sub-tiles are in flight while one is computed.  All four waves compute
// the same S^T = K Q^T (32 keys x 32 rows, the g_q query heads padded to 32) and the same
// softmax statistics; wave w accumulates only d-tile w of O^T += V^T P^T.  The MFMA formulation,
// the swizzled row-major LDS tiles and the transposing V reads are those of the prefill kernel.
//
// Routing (DEC_ROUTE).  Every workgroup of a pair routes by itself: the score rows of the
// pair, their thresholds and the list are computed redundantly, which costs a few
// microseconds of otherwise idle vector and matrix units but no launch, no list in memory and
// no dependent round trip.  Measured (us per step, separate routing and merge launches -> this
// kernel): one sequence of 1000 tokens, 8 kv-heads, 27.6 -> 13.5; 24 of 32k, 2 kv-heads, group of 16 (with a scoring
// launch, see score_in_place in stage2_decode.hip) 76 -> 64; 12 of up to 20000, 8 kv-heads, 83 -> 64.
//
// Merge.  A workgroup writes its partial record and then a flag, both past the caches
// (agent-scope stores), and reads the flags of its pair's splits: whoever sees all of them set
// merges.  Nobody waits; the workgroup whose flag lands last sees them all.  Two that finish at
// the same time may both see all flags and both merge: they write the same values.  The flag
// is a 64-bit number unique to the call, so what the workspace held before cannot be taken for
// a flag (2^-64), and the merging workgroup clears the flags so that a captured launch can be
// replayed with the same number.  (Fencing every partial record device-wide instead writes
// back the L2 once per workgroup: 100 us per step.)
#pragma once
#include <math.h>

#include "common.h"
#include "compress_body.h"
#include "dash_internal.h"
#include "lds_copy.h"
#include "stage1_solve.h"
#include "stage2_args.h"

namespace dash {

enum { DEC_ROUTE = 0, DEC_LISTS = 1, DEC_DENSE = 2 };

struct DecArgs {
  S2Args s;                  // tensors, sizes, part (split partials), seq_lens; mask / bias: the lists to read (DEC_LISTS)
  int splits;                // splits per pair (uniform lengths)
  int slots;                 // splits of a kv-head over the whole batch (per-sequence lengths)
  int batch, n_main;         // n_main: workgroups of the attention; the ones behind update the summary cache
  uint64_t nonce; uint64_t* flags;   // [n_main]
  // Stage 1 (DEC_ROUTE)
  const float* kbar;
  const float* scores; int ld_scores;   // score rows [pair][g_q][ld_scores] of a scoring launch, or null: scored here
  uint32_t* mask_out; float* bias_out; int32_t* cnt; int32_t* idx; float* tau;   // the lists; the last three may be null
  int t_c, window, rows_cap, share_cap;     // LDS sizes: floats of the score area, entries of a split's share
  float xscale, pexp, alpha, inv_sigma;
  float* kbar_upd;           // summary cache to update, or null
};

constexpr int kDecStages = 3;   // LDS ring depth (sub-tiles)

template <int D> struct DecCfg {
  static constexpr int NCH = D / 8;                        // 16-byte chunks per row
  static constexpr int ROW_BYTES = D * 2;
  static constexpr int SUB_BYTES = 32 * ROW_BYTES;         // one 32-key K or V sub-tile
  static constexpr int STAGE_BYTES = 2 * SUB_BYTES;        // K then V
  static constexpr int COPIES = SUB_BYTES / 16 / 256;      // copy instructions per thread, sub-tile and tensor
  static constexpr int ROWS_PER_COPY = 256 / NCH;
  static constexpr size_t RING_BYTES = (size_t)kDecStages * STAGE_BYTES;
  static constexpr int MISC_BYTES = 16;                    // merge decision
};

// same chunk permutations as the prefill tiles (see stage2.hip)
template <int D> __device__ __forceinline__ int dk_swz(int row) {
  return D == 128 ? (row & 15) : ((row >> 1) & 7);
}
template <int D> __device__ __forceinline__ int dv_swz(int row) {
  return D == 128 ? ((row & 3) << 2) : (((row >> 1) & 1) << 2);
}

// ---- scores of 16 chunks ---------------------------------------------------------------------
// x[head][chunk] = xscale <q, kbar> in fp32 on the matrix cores (v_mfma_f32_*_f32: fp32 products
// and sums).  Lane (m = lane % 16, kq = lane / 16) loads d = 16 s + 4 kq .. + 3 of chunk m.
//   groups of up to 4 heads: v_mfma_f32_4x4x1_16b_f32.  Block lane / 4 holds four chunks at one
//     kq, so each of its instructions multiplies 16 chunks x 4 heads at four different d; the
//     four kq partial sums are added through permlane swaps, after which DPP row rho holds the
//     scores of head {0, 2, 1, 3}[rho].
//   groups of 8 and 16: v_mfma_f32_16x16x4_f32, lane (m, kq) receives heads 4 kq .. + 3 of chunk m.
template <int D, bool WIDE> struct DecScore {
  static constexpr int NS = D / 16;
  float qa[NS][4];           // operand A: q[head m % 4 or m][16 s + 4 kq + e], 0 for absent heads
  __device__ __forceinline__ void load_q(const uint16_t* q, int64_t qs_h, int g_q, int lane) {
    const int head = WIDE ? (lane & 15) : (lane & 3), kq = lane >> 4;
    const uint16_t* qp = q + (int64_t)(head < g_q ? head : 0) * qs_h + kq * 4;
#pragma unroll
    for (int s = 0; s < NS; s++) {
      const uint2 w = *reinterpret_cast<const uint2*>(qp + s * 16);
      qa[s][0] = bf16_lo(w.x); qa[s][1] = bf16_hi(w.x); qa[s][2] = bf16_lo(w.y); qa[s][3] = bf16_hi(w.y);
    }
    if (head >= g_q) {
#pragma unroll
      for (int s = 0; s < NS; s++)
#pragma unroll
        for (int e = 0; e < 4; e++) qa[s][e] = 0.f;
    }
  }
  // kbar: the pair's summaries [t_c][D]
  __device__ __forceinline__ void load_tile(const float* kbar, int ct, int n_cand, int lane, f32x4 (&dst)[NS]) const {
    const int c = ct * 16 + (lane & 15);
    const float* kp = kbar + (int64_t)(c < n_cand ? c : n_cand - 1) * D + (lane >> 4) * 4;
#pragma unroll
    for (int s = 0; s < NS; s++) dst[s] = *reinterpret_cast<const f32x4*>(kp + s * 16);
  }
  // dst: [g_q][ld] rows, chunks [0, n_cand) written
  __device__ __forceinline__ void use_tile(const f32x4 (&kv)[NS], int ct, int n_cand, int g_q, float xscale, int lane,
                                           float* dst, int ld) const {
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int s = 0; s < NS; s++)
#pragma unroll
      for (int e = 0; e < 4; e++) {
        if constexpr (WIDE) acc[s & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[s][e], kv[s][e], acc[s & 1], 0, 0, 0);
        else acc[s & 1] = __builtin_amdgcn_mfma_f32_4x4x1f32(qa[s][e], kv[s][e], acc[s & 1], 0, 0, 0);
      }
    f32x4 x;
#pragma unroll
    for (int i = 0; i < 4; i++) x[i] = acc[0][i] + acc[1][i];
    const int m = lane & 15, kq = lane >> 4, c = ct * 16 + m;
    if constexpr (WIDE) {
      if (c < n_cand) {
#pragma unroll
        for (int i = 0; i < 4; i++)
          if (4 * kq + i < g_q) dst[(4 * kq + i) * ld + c] = x[i] * xscale;
      }
    } else {
      typedef uint32_t u2 __attribute__((ext_vector_type(2)));
      const u2 a = __builtin_bit_cast(u2, __builtin_amdgcn_permlane32_swap(__float_as_uint(x[0]), __float_as_uint(x[1]), false, false));
      const u2 b = __builtin_bit_cast(u2, __builtin_amdgcn_permlane32_swap(__float_as_uint(x[2]), __float_as_uint(x[3]), false, false));
      const float y01 = __uint_as_float(a[0]) + __uint_as_float(a[1]);
      const float y23 = __uint_as_float(b[0]) + __uint_as_float(b[1]);
      const u2 w = __builtin_bit_cast(u2, __builtin_amdgcn_permlane16_swap(__float_as_uint(y01), __float_as_uint(y23), false, false));
      const float t = __uint_as_float(w[0]) + __uint_as_float(w[1]);
      const int head = ((kq & 1) << 1) | (kq >> 1);
      if (head < g_q && c < n_cand) dst[head * ld + c] = t * xscale;
    }
  }
};

// agent-scope accesses to the split records (8 bytes at a time): they bypass the caches that
// are not shared by the whole device
__device__ __forceinline__ void agent_store(float* p, float a, float b) {
  const uint64_t w = (uint64_t)__float_as_uint(a) | ((uint64_t)__float_as_uint(b) << 32);
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t agent_load(const void* p) {
  return __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Thresholds and probabilities of this wave's rows (wave, wave + 4, ...), summed over them into
// acc[j] (chunk lane + 64 j).
template <int NJ, int MODE, bool WIDE>
__device__ __forceinline__ void dec_solve(const float* rows, int ld, const DecArgs& a, int n_cand, int wave, int lane,
                                          float* tau_row0 /* this pair's taus, stride n_q = 1, or null */, float (&acc)[NJ]) {
  constexpr int RB = !WIDE ? 1 : (NJ <= 8 ? 4 : 2);
#pragma unroll
  for (int j = 0; j < NJ; j++) acc[j] = 0.f;
  for (int row0 = wave; row0 < a.s.g_q; row0 += 4 * RB) {     // at g_q = 8 two of four rows repeat others
    float v[RB][NJ], tau[RB];
#pragma unroll
    for (int rb = 0; rb < RB; rb++)
#pragma unroll
      for (int j = 0; j < NJ; j++) {
        const int c = lane + 64 * j;
        const int row = RB == 4 ? (row0 + 4 * rb) & (a.s.g_q - 1) : row0 + 4 * rb;
        v[rb][j] = c < n_cand ? rows[row * ld + c] : -INFINITY;
      }
    solve_rows_regs<NJ, RB, MODE>(v, n_cand, a.alpha, a.pexp, tau);
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
      if (RB == 4 && row0 + 4 * rb >= a.s.g_q) break;
#pragma unroll
      for (int j = 0; j < NJ; j++) acc[j] += v[rb][j];
      if (tau_row0 && lane == 0) tau_row0[row0 + 4 * rb] = tau[rb];
    }
  }
}

template <int D, int KIND, int MODE, bool WIDE>
__global__ __launch_bounds__(256, 2) void s2_decode_kernel(DecArgs a) {
  using C = DecCfg<D>;
  constexpr int NST = kDecStages;
  constexpr bool DENSE = KIND == DEC_DENSE, ROUTE = KIND == DEC_ROUTE;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  // the score rows (routing) and the K/V ring (attention) share the first rows_cap floats
  float* rows = reinterpret_cast<float*>(lds);
  float* sbias = rows + a.rows_cap;                              // [share_cap] biases of this split's entries, base 2
  int* xch = reinterpret_cast<int*>(sbias + a.share_cap);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const S2Args& s = a.s;
  const int pairs = s.hb;
  if constexpr (ROUTE) {
    if ((int)blockIdx.x >= a.n_main) {
      // Workgroups behind the attention's: a current token that completes a chunk has that chunk
      // summarised now.  It is the query's own chunk, not a candidate of this step, so no
      // other workgroup reads what is written here.
      const int pr = blockIdx.x - a.n_main, r = pr % s.h_kv, b = pr / s.h_kv;
      const int len = s.seq_lens ? min(max(s.seq_lens[b], 1), s.n_kv) : s.n_kv;
      if (len % s.block != 0) return;
      kbar_block_mean<uint16_t>(s.k, a.kbar_upd, reinterpret_cast<double*>(lds), s.block, D, a.t_c, len / s.block - 1, r, b,
                                s.h_kv, s.ks_b, s.ks_h, s.ks_t);
      return;
    }
  }
  // ---- which pair, which of its ns splits; rec0: record (and flag) of the pair's split 0 ----
  int b, r, split, ns, rec0, len;
  if (!s.seq_lens) {
    // pairs are the fast index: with a multiple of 8 of them all splits of a pair run on one XCD
    const int pair = blockIdx.x % pairs;
    r = pair % s.h_kv; b = pair / s.h_kv;
    split = blockIdx.x / pairs; ns = a.splits; rec0 = pair * ns; len = s.n_kv;
  } else {
    // per-sequence lengths: the slots of a kv-head are dealt to the sequences, at most 64 each (the flags one wave
    // reads)
    const int slots = a.slots;
    r = blockIdx.x % s.h_kv;
    const int slot = blockIdx.x / s.h_kv;
    b = -1; split = 0; ns = 1;
    int first = 0;
    auto chunks_of = [&](int i) { return i < a.batch ? (min(max(s.seq_lens[i], 1), s.n_kv) - 1) / s.block + 1 : 0; };
    // the sequence that `slot` belongs to, from its sequences' shares; share(i) is asked for i = i0 + lane
    auto find = [&](auto&& share) {
      int base = 0;
      for (int i0 = 0; i0 < a.batch && b < 0; i0 += 64) {
        const int cnt = share(i0 + lane);
        int incl = cnt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int t = __shfl_up(incl, o);
          if (lane >= o) incl += t;
        }
        const uint64_t hit = __ballot(base + incl > slot);
        if (hit) {
          const int l = __builtin_ctzll(hit);
          b = i0 + l;
          ns = __builtin_amdgcn_readlane(cnt, l);
          first = base + __builtin_amdgcn_readlane(incl, l) - ns;
        }
        base += __builtin_amdgcn_readlane(incl, 63);
      }
    };
    if constexpr (KIND == DEC_LISTS) {
      // The lists are there, so the slots are dealt by what they say: ceil(sub-tiles / T) each with the smallest
      // T, of 64 that a lane each tries, whose shares fit the slots.  N / (slots - batch) always does.
      // 16 sequences of up to 128k tokens x 8 kv-heads, 9 % of the chunks kept: 139.5 us per step, evenly 146, by
      // length as below 148; a quarter kept: 357, 388, 376; 24 of up to 60000 tokens: 107, 120, 122.
      if (slots == a.batch) {
        b = first = slot;
      } else {
        int* work = reinterpret_cast<int*>(lds);                     // [batch], fewer than 512
        for (int i0 = wave; i0 < a.batch; i0 += 16) {
          uint32_t m[4];
#pragma unroll
          for (int k = 0; k < 4; k++)
            m[k] = i0 + 4 * k < a.batch && lane < s.words ? s.mask[((int64_t)(i0 + 4 * k) * s.h_kv + r) * s.words + lane] : 0u;
#pragma unroll
          for (int k = 0; k < 4; k++) {
            const int i = i0 + 4 * k, kept = (int)wave_sum((float)__popc(m[k]));
            if (i < a.batch && lane == 0) {
              const int end = min(max(s.seq_lens[i], 1), s.n_kv) - 1;
              work[i] = max((kept - 1) * (s.block >> 5) + ((end % s.block) >> 5) + 1, 1);
            }
          }
        }
        __syncthreads();
        float total = 0.f;
        for (int i = lane; i < a.batch; i += 64) total += (float)work[i];
        total = wave_sum(total);
        auto share_at = [&](int i, float inv_t) { return min(max((int)ceilf((float)work[i] * inv_t), 1), 64); };
        const float lo = total / (float)slots, hi = total / (float)(slots - a.batch) + 1.f;
        float inv_t = 1.f / fmaxf(lo + (hi - lo) * (float)lane * (1.f / 63.f), 1.f);
        int sum = 0;
        for (int i = 0; i < a.batch; i++) sum += share_at(i, inv_t);
        const uint64_t fits = __ballot(sum <= slots);
        // (no lane: one split each)
        inv_t = fits ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(inv_t), __builtin_ctzll(fits))) : 0.f;
        find([&](int i) { return i < a.batch ? share_at(i, inv_t) : 0; });
        __syncthreads();                                               // the ring takes the place of `work`
      }
    } else {
      // Half of the slots are dealt evenly (the kept chunks grow more slowly than the length), the others by
      // length: sequence i gets half + floor(extra N_{i+1} / N) - floor(extra N_i / N), N_i = the chunks of the sequences
      // before it, so that no slot is left over
      const int half = max(slots / (2 * a.batch), 1), extra = slots - half * a.batch;
      int tot = 0;
      for (int i0 = 0; i0 < a.batch; i0 += 64) {
        int t = chunks_of(i0 + lane);
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) t += __shfl_xor(t, o);
        tot += t;
      }
      int n_before = 0;
      find([&](int i) {
        const int nc = chunks_of(i);
        int upto = nc;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int t = __shfl_up(upto, o);
          if (lane >= o) upto += t;
        }
        upto += n_before;
        n_before = __builtin_amdgcn_readlane(upto, 63);
        const int share = half + (int)((int64_t)extra * upto / tot) - (int)((int64_t)extra * (upto - nc) / tot);
        return i < a.batch ? min(min(share, 64), nc) : 0;
      });
    }
    if (b < 0) return;                        // more slots than splits
    b = __builtin_amdgcn_readfirstlane(b);
    split = slot - first;
    rec0 = r * slots + first;
    len = min(max(__builtin_amdgcn_readfirstlane(s.seq_lens[b]), 1), s.n_kv);
  }
  const int pair = b * s.h_kv + r;
  const int pos = len - 1;                    // the query's sequence position
  const int cw = pos / s.block;               // its (diagonal) chunk
  const int nsub = s.block >> 5;              // 32-key sub-tiles per chunk

  // ---- Q fragments: rows >= g_q repeat valid heads (their results are dropped); asked for before the list is
  // made, so that the first copies do not wait for them, and behind the scores, which would otherwise wait for them too
  // (a step, against loads in front of the copies, each pair in turn: 1 sequence of 1000 tokens, 32 / 8 heads, 14.2 us ->
  // 13.4, in front of the scores 14.1 -> 13.9; 24 sequences of 32768, 32 / 2 heads, 67.5 -> 66.9, in front of the scores
  // 67.0 -> 67.3).  The list kernels have nothing to overlap them with.
  const int my_head = r * s.g_q + n % s.g_q;
  bf16x8 qf[D / 16];
  auto ask_q = [&]() {
    const uint16_t* qp = s.q + b * s.qs_b + my_head * s.qs_h + h * 8;
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++) qf[ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 16);
  };

  // ---- Stage 1 -------------------------------------------------------------------------------
  uint32_t word = 0u;                         // mask word `lane` of the attended list
  int routed = 0;                             // entries before the local ones (bias 0)
  if constexpr (ROUTE) {
    int n_cand = max(cw - a.window, 0);
    if (n_cand > a.t_c) n_cand = a.t_c;
    const int ld = ((n_cand + 15) >> 4) * 16 + 4;
    const float* xr = rows;
    int xld = ld;
    if (n_cand > 0) {
      if (a.scores) {
        xr = a.scores + (int64_t)pair * s.g_q * a.ld_scores;
        xld = a.ld_scores;
      } else {
        DecScore<D, WIDE> sc;
        const float* kb = a.kbar + (int64_t)pair * a.t_c * D;
        const int nt = (n_cand + 15) >> 4;
        // four tiles in flight per wave: a short row is fetched in one round trip to memory
        f32x4 kv[4][DecScore<D, WIDE>::NS];
#pragma unroll
        for (int i = 0; i < 4; i++)
          if (wave + 4 * i < nt) sc.load_tile(kb, wave + 4 * i, n_cand, lane, kv[i]);
        sc.load_q(s.q + b * s.qs_b + (int64_t)r * s.g_q * s.qs_h, s.qs_h, s.g_q, lane);
        for (int ct = wave; ct < nt; ct += 16) {
#pragma unroll
          for (int i = 0; i < 4; i++) {
            if (ct + 4 * i < nt) {
              sc.use_tile(kv[i], ct + 4 * i, n_cand, s.g_q, a.xscale, lane, rows, ld);
              if (ct + 4 * i + 16 < nt) sc.load_tile(kb, ct + 4 * i + 16, n_cand, lane, kv[i]);
            }
          }
        }
      }
      __syncthreads();
      // one row per wave at a time; the probabilities of a wave's rows are summed in registers,
      // those of the four waves through LDS (the score rows are dead by then)
      float* tau0 = (a.tau && split == 0) ? a.tau + (int64_t)b * s.h_q + r * s.g_q : nullptr;
      const int nj = (n_cand + 63) >> 6;
#define DASH_DEC_SOLVE(NJ_)                                                            \
  {                                                                                    \
    float acc[NJ_];                                                                    \
    dec_solve<NJ_, MODE, WIDE>(xr, xld, a, n_cand, wave, lane, tau0, acc);             \
    __syncthreads();                                                                   \
    _Pragma("unroll") for (int j = 0; j < NJ_; j++)                                    \
      if (lane + 64 * j < n_cand) rows[wave * ld + lane + 64 * j] = acc[j];            \
  }
      if (nj <= 1) DASH_DEC_SOLVE(1)
      else if (nj <= 2) DASH_DEC_SOLVE(2)
      else if (nj <= 4) DASH_DEC_SOLVE(4)
      else if (nj <= 8) DASH_DEC_SOLVE(8)
      else if (nj <= 16) DASH_DEC_SOLVE(16)
      else DASH_DEC_SOLVE(32)
#undef DASH_DEC_SOLVE
    } else if (a.tau && split == 0 && tid < s.g_q) {
      a.tau[(int64_t)b * s.h_q + r * s.g_q + tid] = 0.f;
    }
    ask_q();
    __syncthreads();
    // Group weights and membership.  Every wave goes through all 64-chunk slots by itself: the
    // mask words (lane i holds word i) and the counts then need no exchange.
    const float inv_g = 1.f / (float)s.g_q;
    auto weight = [&](int c) {
      return c < n_cand ? ((rows[c] + rows[ld + c]) + (rows[2 * ld + c] + rows[3 * ld + c])) * inv_g : 0.f;
    };
    // ln via the hardware log2 (about 1 ulp): ample for a bias that is divided by sigma
    auto ln = [](float w) { return __builtin_amdgcn_logf(w) * 0.6931471805599453f; };
    float slog = 0.f;
    const int nslot = (n_cand + 63) >> 6;
#pragma unroll 2
    for (int j = 0; j < nslot; j++) {
      const float w = weight(lane + 64 * j);
      const uint64_t bal = __ballot(w > 0.f);
      if (w > 0.f) slog += ln(w);
      if ((lane >> 1) == j) word = (lane & 1) ? (uint32_t)(bal >> 32) : (uint32_t)bal;
      routed += __popcll(bal);
    }
    slog = wave_sum(slog);
    const float mu = routed > 0 ? slog / (float)routed : 0.f;
    const int c0 = max(cw - a.window, 0);     // the local set: window chunks, then the own chunk
    const int total = routed + cw - c0 + 1;
    const int nt_all = (total - 1) * nsub + ((pos - cw * s.block) >> 5) + 1;
    const int per = (nt_all + ns - 1) / ns;
    const int e0 = split * per / nsub, e1 = min((min(split * per + per, nt_all) + nsub - 1) / nsub, total);
    // ids and biases of this split's entries, into the lists too.  The slots are dealt to the waves; an entry cut
    // between two splits is written by both, with the same values.
    int32_t* oidx = a.idx ? a.idx + (int64_t)pair * s.t_all : nullptr;
    float* obias = a.bias_out + (int64_t)pair * s.t_all;
    int start = 0;
    for (int j = 0; j < nslot; j++) {
      const uint32_t lo = __builtin_amdgcn_readlane(word, 2 * j), hi = __builtin_amdgcn_readlane(word, 2 * j + 1);
      const uint64_t bal = (uint64_t)lo | ((uint64_t)hi << 32);
      const int cnt = __popcll(bal);
      if ((j & 3) == wave && start < e1 && start + cnt > e0 && ((bal >> lane) & 1u)) {
        const int p = start + __popcll(bal & ((1ull << lane) - 1ull));
        if (p >= e0 && p < e1) {
          const float d = (ln(weight(lane + 64 * j)) - mu) * a.inv_sigma;
          sbias[p - e0] = d * kLog2e;
          obias[p] = d;
          if (oidx) oidx[p] = lane + 64 * j;
        }
      }
      start += cnt;
    }
    for (int c = c0; c <= cw; c++)            // at most 9 local chunks
      if (lane == (c >> 5)) word |= 1u << (c & 31);
    if (tid <= cw - c0) {
      const int p = routed + tid;
      if (p >= e0 && p < e1) {
        sbias[p - e0] = 0.f;
        obias[p] = 0.f;
        if (oidx) oidx[p] = c0 + tid;
      }
    }
    if (split == 0 && a.cnt && tid == 0) a.cnt[pair] = total;
    if (split == 0 && tid < s.words) a.mask_out[(int64_t)pair * s.words + tid] = word;
    __syncthreads();                          // the score rows give way to the K / V ring
  }

  // ---- this workgroup's share of the attended list -------------------------
  // lane i holds mask word i; `total` entries in ascending order, the diagonal chunk last; its
  // sub-tiles end with the query's own key.  Sub-tiles [t0, t1) of the list are ours.
  int total, incl = 0;
  if (DENSE) {
    total = (s.causal ? cw : s.t_all - 1) + 1;
  } else {
    if (!ROUTE && lane < s.words) word = s.mask[(int64_t)pair * s.words + lane];
    incl = __popc(word);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int t = __shfl_up(incl, off);
      if (lane >= off) incl += t;
    }
    total = __builtin_amdgcn_readlane(incl, 63);
  }
  const int last_sub = s.causal ? ((pos - cw * s.block) >> 5) + 1 : nsub;
  const int nt_all = (total - 1) * nsub + last_sub;
  const int per = (nt_all + ns - 1) / ns;
  const int t0 = split * per, t1 = min(nt_all, t0 + per);
  const int e0 = t0 / nsub;
  float* part = s.part + ((int64_t)(rec0 + split) * s.g_q) * (D + 2);

  // online-softmax state (base-2 logits)
  float m_run = -INFINITY, l_run = 0.f;
  f32x16 oacc;
#pragma unroll
  for (int j = 0; j < 16; j++) oacc[j] = 0.f;

  if (t0 < t1) {
    if (KIND == DEC_LISTS) {
      // the diagonal chunk (last entry of a causal list) carries bias 0
      const int e1 = (t1 + nsub - 1) / nsub;
      const float* bl = s.bias + (int64_t)pair * s.t_all;
      for (int e = e0 + tid; e < e1; e += 256) sbias[e - e0] = s.causal && e == total - 1 ? 0.f : bl[e] * kLog2e;
    }
    // chunk-id iterator over the mask, positioned at entry e0 (wave-uniform scalars)
    int it_wi = 0;
    uint32_t it_bits = 0u;
    if (!DENSE) {
      // first word whose inclusive count exceeds e0
      const uint64_t ball = __ballot(incl > e0);
      it_wi = __builtin_ctzll(ball);
      const int before = __builtin_amdgcn_readlane(incl, it_wi) - __popc(__builtin_amdgcn_readlane(word, it_wi));
      it_bits = __builtin_amdgcn_readlane(word, it_wi);
      for (int i = before; i < e0; i++) it_bits &= it_bits - 1u;   // drop the entries below e0
    }
    int it_e = e0;   // entry the iterator points at
    auto next_id = [&]() -> int {   // id of entry it_e, then advance
      int id;
      if (DENSE) {
        id = it_e;
      } else {
        while (it_bits == 0u) { it_wi++; it_bits = __builtin_amdgcn_readlane(word, it_wi); }
        id = it_wi * 32 + __builtin_ctz(it_bits);
        it_bits &= it_bits - 1u;
      }
      it_e++;
      return id;
    };

    if constexpr (!ROUTE) ask_q();
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++) asm volatile("" : "+v"(qf[ks]));   // loads done before the copies are in flight

    // ---- global -> LDS sub-tile copies (layout as in the prefill kernel) -------
    const u32x4 k_rs = make_rsrc(s.k + b * s.ks_b + r * s.ks_h, (((int64_t)len - 1) * s.ks_t + D) * 2);
    const u32x4 v_rs = make_rsrc(s.v + b * s.vs_b + r * s.vs_h, (((int64_t)len - 1) * s.vs_t + D) * 2);
    const uint32_t lds0 = lds_addr_of(lds);
    const int c_row = (wave * 64 + lane) / C::NCH, c_pos = lane % C::NCH;
    const uint32_t k_off = (uint32_t)(c_row * (int)s.ks_t * 2 + ((c_pos ^ dk_swz<D>(c_row)) << 4));
    const uint32_t v_off = (uint32_t)(c_row * (int)s.vs_t * 2 + ((c_pos ^ dv_swz<D>(c_row)) << 4));
    const uint32_t k_step = (uint32_t)(C::ROWS_PER_COPY * (int)s.ks_t * 2);
    const uint32_t v_step = (uint32_t)(C::ROWS_PER_COPY * (int)s.vs_t * 2);
    const int n_sub = t1 - t0;   // sub-tiles this workgroup streams
    int cp_t = 0, cp_sub = t0 - e0 * nsub, cp_id = next_id();
    auto copy_next = [&]() {   // sub-tile cp_t -> ring slot cp_t % NST
      const uint32_t dst = lds0 + (cp_t % NST) * C::STAGE_BYTES + wave * 1024;
      const uint32_t key0 = (uint32_t)(cp_id * s.block + cp_sub * 32);
      const uint32_t tk = key0 * (uint32_t)s.ks_t * 2u, tv = key0 * (uint32_t)s.vs_t * 2u;
#pragma unroll
      for (int i = 0; i < C::COPIES; i++) copy16_to_lds(k_rs, dst + i * 4096, k_off, tk + i * k_step);
#pragma unroll
      for (int i = 0; i < C::COPIES; i++) copy16_to_lds(v_rs, dst + C::SUB_BYTES + i * 4096, v_off, tv + i * v_step);
      cp_t++;
      if (++cp_sub == nsub) { cp_sub = 0; if (cp_t < n_sub) cp_id = next_id(); }
    };
    // ---- operand read addresses (bytes inside a ring slot) -----------------------
    uint32_t k_rd[D / 16];
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++)
      k_rd[ks] = (uint32_t)(n * C::ROW_BYTES + (((2 * ks + h) ^ dk_swz<D>(n)) << 4));
    const int s16 = lane & 15, a16 = (lane >> 4) & 1;
    const int dtile = wave < D / 32 ? wave : 0;   // the d-tile this wave accumulates
    const uint32_t v_rd = (uint32_t)(C::SUB_BYTES + (4 * h + (s16 >> 2)) * C::ROW_BYTES +
                                     ((((4 * dtile) ^ dv_swz<D>(s16 >> 2)) + 2 * a16 + ((s16 & 3) >> 1)) << 4) +
                                     ((s16 & 1) << 3));

    // ---- prologue: NST - 1 sub-tiles in flight ---------------------------------
#pragma unroll
    for (int i = 0; i < NST - 1; i++)
      if (i < n_sub) copy_next();

    // ---- main loop ---------------------------------------------------------------
    // Iteration t: wait until this wave's copies of sub-tile t have landed (all but
    // the newest NST - 2 sub-tiles' worth of copies; everything once the last
    // sub-tile has been issued), barrier (everybody's copies visible; sub-tile
    // t - 1 no longer read), start the copy of sub-tile t + NST - 1 into the slot
    // of sub-tile t - 1, compute sub-tile t.
    int e_c = e0, sub_c = t0 - e0 * nsub;
    for (int t = 0; t < n_sub; t++) {
      if (cp_t - t - 1 >= NST - 2) {
        static_assert(NST == 3, "the wait below counts one sub-tile's copies");
        if constexpr (C::COPIES == 2) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
      } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      __syncthreads();
      if (cp_t < n_sub) copy_next();
      const float bias_c = DENSE ? 0.f : sbias[e_c - e0];

      const char* sb = lds + (t % NST) * C::STAGE_BYTES;
      f32x16 sc;
      {
        bf16x8 kf[D / 16];
#pragma unroll
        for (int ks = 0; ks < D / 16; ks++) kf[ks] = *reinterpret_cast<const bf16x8*>(sb + k_rd[ks]);
        const f32x16 z = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0], qf[0], z, 0, 0, 0);
#pragma unroll
        for (int ks = 1; ks < D / 16; ks++) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], sc, 0, 0, 0);
      }
      // V^T fragments of this wave's d-tile (contraction steps g = 0, 1)
      bf16x8 vf[2];
      if (wave < D / 32) {
#pragma unroll
        for (int g = 0; g < 2; g++)
          vf[g] = lds_read_tr_pair(sb + v_rd + (16 * g) * C::ROW_BYTES, sb + v_rd + (16 * g + 8) * C::ROW_BYTES);
      }
      // dead keys: after the query's position (diagonal chunk), past the end of the sequence
      // (the ragged last chunk of a non-causal dense call)
      if (e_c == total - 1) {
        const int chunk = s.causal ? cw : e_c;
        const int lim = (s.causal ? pos : s.n_kv - 1) - (chunk * s.block + sub_c * 32 + 4 * h);   // dead if c > lim
#pragma unroll
        for (int j = 0; j < 16; j++) {
          const int c = (j >> 2) * 8 + (j & 3);
          sc[j] = c > lim ? -INFINITY : sc[j];
        }
      }
      float mloc = -INFINITY;
#pragma unroll
      for (int j = 0; j < 16; j += 2) mloc = fmaxf(fmaxf(mloc, sc[j]), sc[j + 1]);
      mloc = fmaxf(mloc, __shfl_xor(mloc, 32));
      const float tmax = fmaf(mloc, s.c1, bias_c);
      // lazy rescaling: see the prefill kernel
      if (__any(tmax > m_run + kLazy)) {
        const float m_new = fmaxf(m_run, tmax);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;
        const float corr = __builtin_amdgcn_exp2f(m_run - m_use);
        m_run = m_new;
        l_run *= corr;
#pragma unroll
        for (int j = 0; j < 16; j++) oacc[j] *= corr;
      }
      const float off = bias_c - (m_run == -INFINITY ? 0.f : m_run);
      u32x4 pb[2];
      float lsum = 0.f;
#pragma unroll
      for (int j = 0; j < 16; j += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[j], s.c1, off));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(sc[j + 1], s.c1, off));
        lsum += p0 + p1;
        const bf16x2 w2 = {(__bf16)p0, (__bf16)p1};
        pb[j >> 3][(j & 7) >> 1] = __builtin_bit_cast(uint32_t, w2);
      }
      l_run += lsum;
      if (wave < D / 32) {
#pragma unroll
        for (int g = 0; g < 2; g++)
          oacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[g], __builtin_bit_cast(bf16x8, pb[g]), oacc, 0, 0, 0);
      }
      if (++sub_c == nsub) { sub_c = 0; e_c++; }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no copy may outlive the workgroup's LDS
  }

  const float l_tot = l_run + __shfl_xor(l_run, 32);
  if (ns == 1) {
    // the whole list was ours
    if (n < s.g_q && wave < D / 32) {
      const float inv = 1.f / l_tot;
      uint16_t* op = s.o + b * s.os_b + (int64_t)(r * s.g_q + n) * s.os_h + wave * 32 + h * 4;
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        uint2 w;
        w.x = pack_bf16x2(oacc[q4 * 4 + 0] * inv, oacc[q4 * 4 + 1] * inv);
        w.y = pack_bf16x2(oacc[q4 * 4 + 2] * inv, oacc[q4 * 4 + 3] * inv);
        *reinterpret_cast<uint2*>(op + q4 * 8) = w;
      }
    }
    return;
  }
  // ---- partial record per (split, head-in-group): D floats of unnormalised O, then the
  // running max (base-2 logits) and the running sum; an empty share has max -inf, sum 0 -------
  if (n < s.g_q) {
    float* pp = part + n * (D + 2);
    if (wave < D / 32) {
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        float* pq = pp + wave * 32 + q4 * 8 + h * 4;
        agent_store(pq, oacc[q4 * 4 + 0], oacc[q4 * 4 + 1]);
        agent_store(pq + 2, oacc[q4 * 4 + 2], oacc[q4 * 4 + 3]);
      }
    }
    if (wave == 0 && h == 0) agent_store(pp + D, m_run, l_tot);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the record is in memory ...
  __syncthreads();
  if (wave == 0) {
    uint64_t* fl = a.flags + rec0;
    if (lane == 0) __hip_atomic_store(fl + split, a.nonce, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // ... before the flag, and the flag before the flags are read
    uint64_t f = a.nonce;
    if (lane < ns) f = agent_load(fl + lane);
    const bool all = __all(f == a.nonce);
    if (lane == 0) *xch = all;
  }
  __syncthreads();
  if (!*xch) return;

  // ---- merge: o = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s ------------------------------
  // The weights of all (split, head) first (each record's max and sum, one round trip), then
  // every thread sums 4 d of a head over the splits, SB records in flight.
  float* wts = rows;                          // [ns][g_q] weights / denominator
  const float* rec = s.part + (int64_t)rec0 * s.g_q * (D + 2);
  float* mls = wts + 64 * 16;                 // [ns][g_q][2] maxima and sums
  for (int i = tid; i < ns * s.g_q; i += 256) {
    const uint64_t ml = agent_load(rec + (int64_t)i * (D + 2) + D);
    mls[2 * i] = __uint_as_float((uint32_t)ml);
    mls[2 * i + 1] = __uint_as_float((uint32_t)(ml >> 32));
  }
  constexpr int SB = 4, HP = D / 4;
  __syncthreads();
  for (int i = tid; i < ns * s.g_q; i += 256) {
    const int head = i % s.g_q;
    float M = -INFINITY, den = 0.f;
    for (int k = 0; k < ns; k++) M = fmaxf(M, mls[2 * (k * s.g_q + head)]);
    for (int k = 0; k < ns; k++) den = fmaf(__builtin_amdgcn_exp2f(mls[2 * (k * s.g_q + head)] - M), mls[2 * (k * s.g_q + head) + 1], den);
    wts[i] = __builtin_amdgcn_exp2f(mls[2 * i] - M) / den;
  }
  __syncthreads();
  for (int it = tid; it < s.g_q * HP; it += 256) {
    const int head = it / HP, d4 = (it % HP) * 4;
    const float* ph = rec + head * (D + 2) + d4;
    float o4[4] = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < ns; s0 += SB) {
      uint64_t ov[SB][2];
#pragma unroll
      for (int i = 0; i < SB; i++) {
        const float* ps = ph + (int64_t)min(s0 + i, ns - 1) * s.g_q * (D + 2);
        ov[i][0] = agent_load(ps);
        ov[i][1] = agent_load(ps + 2);
      }
#pragma unroll
      for (int i = 0; i < SB; i++) {
        const float w = s0 + i < ns ? wts[(s0 + i) * s.g_q + head] : 0.f;
#pragma unroll
        for (int e = 0; e < 4; e++) o4[e] = fmaf(w, __uint_as_float((uint32_t)(ov[i][e >> 1] >> (32 * (e & 1)))), o4[e]);
      }
    }
    uint2 w;
    w.x = pack_bf16x2(o4[0], o4[1]);
    w.y = pack_bf16x2(o4[2], o4[3]);
    *reinterpret_cast<uint2*>(s.o + b * s.os_b + (int64_t)(r * s.g_q + head) * s.os_h + d4) = w;
  }
  if (tid < ns) __hip_atomic_store(a.flags + rec0 + tid, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace dash
