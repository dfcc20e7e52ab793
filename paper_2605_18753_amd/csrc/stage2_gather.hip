// Stage 2 (bf16 prefill) where tokens keep few chunks: every chunk is attended by the rows that kept it, gathered.
//
// The kernel of stage2.hip walks the union of 128 rows' chunks and multiplies a wave's 32 rows with every chunk that one of
// its tokens kept.  Where tokens keep a tenth of the chunks, each for itself, the union of eight tokens holds
// six tenths and a workgroup's nearly all.  Here a workgroup (8 waves) owns 256 (token, head) rows with their output sums in LDS (fp32,
// 128 KB at head dimension 128), and a wave takes one item at a time: a chunk and up to 32 / g_q tokens that kept it.  The rows of those
// tokens are gathered into two tiles of 16 columns, the chunk's keys and values come from L2 straight into
// registers (nobody else in the workgroup needs them), and the item's sums are added to the rows' in LDS.
//
// Items are numbered chunk by chunk, and a wave takes the next number (LDS counter).  It adds its sums once every token's earlier list
// entries are in (LDS, per token), so that the result does not depend on which wave was faster.  A wave waits for items with smaller numbers only,
// and the number it takes before it adds is larger than the one it holds: the smallest outstanding item never waits.  With one order for all items instead
// of one per token the waves queued at the sums: 68 -> 46 ms for 128k tokens in chunks of 128.
//
// v_mfma_f32_16x16x32_bf16, lane (m = lane % 16, kq = lane / 16):
//   S^T[key,row] = K Q^T    A = K: lane (m, kq) holds key m, 8 d of step s; B = Q: row m, the same d
//   accumulator: lane (m, kq) holds row m, keys 4 kq + 0..3: two key tiles give the 8 contraction slots of lane (m, kq) in
//   O^T[d,row] += V^T P^T   A = V^T: lane (m, kq) loads D/16 consecutive d (from D/16 m) of its 8 keys and pairs the keys up with byte
//   permutes, one per operand register; accumulator e, register r of lane (m, kq) is d = (4 kq + r) D/16 + e of row m.
// The A and B operands want adjacent lanes on different rows of K and Q, for which the memory pipe takes 64 accesses an instruction, one a
// clock: 3250 of them per item instead of 1340.  So four adjacent lanes load 64 bytes of a row, and the LDS crossbar moves them to their lanes (with
// selects between neighbouring lanes instead the vector pipe has 27 % more to do: 3.20 -> 3.10 ms at 32k tokens, group of 4, 9 % kept).
//
// What bounds it: a wave's chain of loads, products and vector work, two waves per SIMD (256 registers and twelve to fifteen spilled, most of
// them reloaded once per item; head dimension 64: three waves, none spilled, 1.97 -> 1.79 ms there).  128k tokens, 32 / 8 heads, chunks of 128, 12 % of them kept:
// 87 -> 40 ms for Stage 2 alone, vector pipe two fifths and matrix pipe a fifth busy, 20 TB/s out of L2.  Copies without one part: no loads but an item's first -18 %, no sums in LDS -10, no wait for a token's earlier entries -7
// (before tiles were added one by one), no exponentials -2.
#include <type_traits>

#include "common.h"
#include "dash_internal.h"
#include "lds_copy.h"
#include "stage2_args.h"

namespace dash {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Launches of fewer 128-row tiles times 64-key tiles of a row (half of them for a whole causal prompt) are not looked at, so that no launch under
// 1 ms pays for finding out what the lists hold and for the launch not used: 6 to 12 us (4096 tokens, 32 / 8 heads, dense 160 -> 167 us; 8192, 43 % kept,
// 483 -> 494; 12000, a third kept, 974 -> 985; at 32k tokens, 7.7 ms, 13 us).  The line is drawn for the launches that stay, and those below it that
// the costs would send here are left out.  Stage 2, there -> here: 2000 tokens against a 32k cache (249k of these) with 12 % kept 681 -> 414 us, 20 % 803 -> 598, correlated
// queries and 2.5 % 199 -> 174, head dimension 64 and 12 % 498 -> 246; 8192 tokens, 32 / 8 heads (131k), 12 % 356 -> 284; 16000 tokens of 16 heads (250k), 8 % 829 -> 511.
constexpr int64_t kMinTiles = 320000;

template <int D, int G> struct GatherCfg {
  static constexpr int ROWS = 256, TOK = ROWS / G, TPI = 32 / G;   // rows and tokens of a workgroup, tokens of an item
  static constexpr int WAVES = D == 64 ? 12 : 8;
  static constexpr int TOKP = TOK + 1;                             // row stride of the mask words: no bank conflicts
  static size_t lds_bytes(int words) {
    return (size_t)ROWS * D * 4 + 2 * ROWS * 4 + (size_t)words * TOKP * 4 + (((size_t)words * TOKP * 2 + 3) & ~(size_t)3) + words * 32 * 2 + 16 + TOK * 4;
  }
};

template <int D, int G>
__global__ __launch_bounds__((GatherCfg<D, G>::WAVES * 64), (GatherCfg<D, G>::WAVES / 4)) void s2_gather_kernel(S2Args a) {
  using C = GatherCfg<D, G>;
  constexpr int TOK = C::TOK, TPI = C::TPI, TOKP = C::TOKP;
  constexpr int NE = D / 16;            // accumulators of a 16-row tile
  constexpr int NS = D / 32;            // contraction steps of the first product
  constexpr int NW = TOK > 64 ? TOK / 64 : 1;   // 64 tokens per lane step
  constexpr int NB = D / 16;            // 16-byte pieces of a row's sums per lane
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  f32x4* lo = reinterpret_cast<f32x4*>(lds);                              // [NB][4][256]: piece j, quarter kq, row
  float* lm = reinterpret_cast<float*>(lds + C::ROWS * D * 4);            // [256] reference maxima
  float* ll = lm + C::ROWS;                                               // [256] sums
  uint32_t* lmask = reinterpret_cast<uint32_t*>(ll + C::ROWS);            // [words][TOKP] mask words
  uint16_t* lpre = reinterpret_cast<uint16_t*>(lmask + a.words * TOKP);   // [words][TOKP] list entries before the word
  uint16_t* lcum = reinterpret_cast<uint16_t*>(lmask + a.words * TOKP + (a.words * TOKP + 1) / 2);   // [words * 32] items up to and with the chunk
  int* ctl = reinterpret_cast<int*>(lcum + a.words * 32);                 // next item, choice
  int* ldone = ctl + 4;                                                   // [TOK] list entries of a token that are in

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 15, kq = lane >> 4;
  const int bid = blockIdx.x;
  const int hbi = bid % a.hb;
  const int blk = (a.n_tiles + 1) / 2 - 1 - bid / a.hb;                   // longest rows first
  const int r = hbi % a.h_kv, b = hbi / a.h_kv;
  // Workgroups dispatched together (256, one per CU) begin their walks together: the 32 of a die read the same head's chunks at the same
  // time, out of its L2 (128k tokens in chunks of 128: L2 misses 6.8 % of the requests -> 4.7, 38.5 -> 38.4 ms for Stage 2; chunks of 64 17.49 -> 17.54,
  // 32k tokens 2.08 -> 2.09: by now it is worth nothing where a head fits the L2, and little where it does not).
  int* arrived = a.choice->arrived + (bid & 7) * 32;
  if (wave == 0) {                                                        // one wave asks: what the record says may change between two looks
    const int c = s2_choice(a, lane);
    if (lane == 0) ctl[1] = c;
  }
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(ctl[1]) < 0) return;                 // s2_attend_kernel has attended
  if (tid == 0) __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int tok0 = blk * TOK;
  const int n_tok = min(TOK, a.n_q - tok0);
  const int64_t row0 = ((int64_t)b * a.h_kv + r) * a.n_q + tok0;
  const int block_log = 31 - __builtin_clz(a.block);
  const int wn = a.words;

  for (int i = tid; i < TOK * wn; i += C::WAVES * 64) {
    const int t = i / wn, w = i - t * wn;
    lmask[w * TOKP + t] = t < n_tok ? a.mask[(row0 + t) * a.words + w] : 0u;
  }
  for (int i = tid; i < C::ROWS * D / 4; i += C::WAVES * 64) lo[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (tid < 256) { lm[tid] = -INFINITY; ll[tid] = 0.f; }
  if (tid == 0) ctl[0] = 0;
  if (tid < TOK) ldone[tid] = 0;
  __syncthreads();
  for (int w = wave; w < wn; w += C::WAVES) {
    uint32_t v[NW];
#pragma unroll
    for (int k = 0; k < NW; k++) {
      v[k] = lane < TOK ? lmask[w * TOKP + 64 * k + lane] : 0u;
      if (lane < TOK) lpre[w * TOKP + 64 * k + lane] = (uint16_t)__popc(v[k]);
    }
    int items = 0;
#pragma unroll 2
    for (int i = 0; i < 32; i++) {
      int n = 0;
#pragma unroll
      for (int k = 0; k < NW; k++) n += __popcll(__ballot((v[k] >> i) & 1u));
      items = lane == i ? (n + TPI - 1) / TPI : items;
    }
    if (lane < 32) lcum[w * 32 + lane] = (uint16_t)items;
  }
  __syncthreads();
  if (wave == 0) {
    int base = 0;
    for (int c = lane; c - lane < wn * 32; c += 64) {
      const int incl = base + wave_scan(c < wn * 32 ? lcum[c] : 0);
      if (c < wn * 32) lcum[c] = (uint16_t)incl;
      base = __builtin_amdgcn_readlane(incl, 63);
    }
  } else if (tid - 64 < TOK) {
    int run = 0;
    for (int w = 0; w < wn; w++) {
      const int x = lpre[w * TOKP + tid - 64];
      lpre[w * TOKP + tid - 64] = (uint16_t)run;
      run += x;
    }
  }
  __syncthreads();
  const int n_items = lcum[wn * 32 - 1];
  if (tid == 0) {
    // never more than about a twentieth of the walk's time: the others may not get a CU for as long as this one runs
    const int all = (min((bid | 255) + 1, (int)gridDim.x) - (bid & 7) + 7) >> 3;
    for (int i = 0; i < n_items >> 5 && __hip_atomic_load(arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < all; i++)
      __builtin_amdgcn_s_sleep(16);
  }
  __syncthreads();

  auto rsrc = [](const void* p, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (uint32_t)bytes, 0x00020000);
  };
  const __amdgpu_buffer_rsrc_t q_rs = rsrc(a.q + b * a.qs_b + (int64_t)r * G * a.qs_h, ((int64_t)(G - 1) * a.qs_h + (int64_t)(a.n_q - 1) * a.qs_t + D) * 2);
  const __amdgpu_buffer_rsrc_t k_rs = rsrc(a.k + b * a.ks_b + r * a.ks_h, ((int64_t)(a.n_kv - 1) * a.ks_t + D) * 2);
  const __amdgpu_buffer_rsrc_t v_rs = rsrc(a.v + b * a.vs_b + r * a.vs_h, ((int64_t)(a.n_kv - 1) * a.vs_t + D) * 2);
  const __amdgpu_buffer_rsrc_t b_rs = rsrc(a.bias + row0 * a.t_all, (int64_t)n_tok * a.t_all * 4);
  const uint32_t ks2 = (uint32_t)a.ks_t * 2u, vs2 = (uint32_t)a.vs_t * 2u;
  // K and Q: lane l loads piece l % 4 of the 64 bytes of step s of row l / 4, and the LDS crossbar hands lane (m, kq) what lane 4 m + kq loaded
  const uint32_t k_off = (uint32_t)(lane >> 2) * ks2 + (uint32_t)(lane & 3) * 16u;
  const int from = (4 * m + kq) * 4;
  auto turn = [&](bf16x8 (&f)[NS]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < NS; s++) {
      u32x4 x = __builtin_bit_cast(u32x4, f[s]);
#pragma unroll
      for (int w = 0; w < 4; w++) x[w] = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)x[w]);
      f[s] = __builtin_bit_cast(bf16x8, x);
    }
  };
  const uint32_t v_off = (uint32_t)(4 * kq) * vs2 + (uint32_t)m * (D / 8u);
  constexpr int VW = D / 32;            // registers of a value load

  // ---- the item in hand --------------------------------------------------------
  bf16x8 qf[2][NS];
  bf16x8 kf[2][NS];
  uint32_t vr[8][VW];
  float bias[2], m_ref[2], l[2] = {0.f, 0.f};
  int tag[2] = {-1, -1};                // row of the workgroup's, list entry of its token << 8; -1: no token
  int chunk = 0, cb = 0;
  bool two = false;
  f32x4 acc[2][NE];

  auto load_k = [&](int key0) {
#pragma unroll
    for (int kt = 0; kt < 2; kt++) {
#pragma unroll
      for (int s = 0; s < NS; s++)
        kf[kt][s] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(k_rs, k_off + s * 64, (uint32_t)(key0 + 16 * kt) * ks2, 0));
    }
  };
  auto load_v = [&](int key0) {
#pragma unroll
    for (int i = 0; i < 8; i++) {
      const uint32_t so = (uint32_t)(key0 + (i & 3) + (i >> 2) * 16) * vs2;
      if constexpr (D == 128) {
        const u32x4 x = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(v_rs, v_off, so, 0));
#pragma unroll
        for (int e = 0; e < 4; e++) vr[i][e] = x[e];
      } else {
        const u32x2 x = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(v_rs, v_off, so, 0));
        vr[i][0] = x[0]; vr[i][1] = x[1];
      }
    }
  };
  auto set_up = [&](int item) __attribute__((always_inline)) {
    int at;
    for (;;) {
      const int x = cb + lane < wn * 32 ? (int)lcum[cb + lane] : 0x7fffffff;
      const uint64_t le = __ballot(x <= item);
      at = __popcll(le);
      if (at < 64) break;
      cb += 64;
    }
    chunk = cb + at;
    const int sub = item - (chunk > 0 ? __builtin_amdgcn_readfirstlane((int)lcum[max(chunk - 1, 0)]) : 0);
    const int w = chunk >> 5, bi = chunk & 31;
    // the chunk's tokens TPI sub .. + TPI - 1 go to lanes 0 .. TPI - 1; whoever is not among them pushes to the last lane
    int cnt = 0, tok_of = 0;
#pragma unroll
    for (int k = 0; k < NW; k++) {
      const uint32_t mv = lmask[w * TOKP + 64 * k + min(lane, TOK - 1)];
      const int pre = lpre[w * TOKP + 64 * k + min(lane, TOK - 1)];
      const bool bit = lane < TOK && ((mv >> bi) & 1u);
      const uint64_t set = __ballot(bit);
      const int to = cnt - sub * TPI + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(set >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)set, 0u));
      const int entry = pre + __popc(mv & ((1u << bi) - 1u));
      const int x = __builtin_amdgcn_ds_permute((bit && to >= 0 && to < TPI ? to : 63) * 4, (64 * k + lane) * G | entry << 8);
      tok_of = k == 0 || sub * TPI + lane >= cnt ? x : tok_of;
      cnt += __popcll(set);
    }
    const int n_in = cnt - sub * TPI;            // of the item and those behind it
    two = n_in > TPI / 2;
    uint32_t qo[2];
#pragma unroll
    for (int j = 0; j < 2; j++) {
      const int slot = j * (TPI / 2) + m / G, qs = j * (TPI / 2) + (lane >> 2) / G;   // of the lane's row, of the row it loads
      const int x = __builtin_amdgcn_ds_bpermute(slot * 4, tok_of), xq = __builtin_amdgcn_ds_bpermute(qs * 4, tok_of);
      const bool ok = slot < n_in;
      tag[j] = ok ? x + m % G : -1;
      const int t = ok ? (x & 0xff) / G : 0;
      qo[j] = qs < n_in ? (uint32_t)((lane >> 2) % G * (int)a.qs_h + (tok0 + (xq & 0xff) / G) * (int)a.qs_t + (lane & 3) * 8) * 2u : 0x80000000u;
      const bool own = a.causal && chunk == (a.pos0 + tok0 + t) >> block_log;
      // read past the end: 0
      bias[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(b_rs, ok && !own ? (uint32_t)(t * a.t_all + (x >> 8)) * 4u : ~3u, 0, 0));
    }
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int s = 0; s < NS; s++)
        qf[j][s] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(q_rs, qo[j] + s * 64, 0, 0));
    load_k(chunk << block_log);
    load_v(chunk << block_log);
  };

  auto attend = [&](auto nt_tag) __attribute__((always_inline)) {
    constexpr int NT = decltype(nt_tag)::value;
    bool edge = false;
    int lim[NT];
#pragma unroll
    for (int j = 0; j < NT; j++) {
      bias[j] = tag[j] < 0 ? -INFINITY : bias[j] * kLog2e;
      // the last key a row may see: its own in its own chunk, else the sequence's last
      const int pos = a.pos0 + tok0 + (tag[j] & 0xff) / G;
      lim[j] = a.causal && chunk == pos >> block_log ? pos : a.n_kv - 1;
      edge |= tag[j] >= 0 && ((chunk + 1) << block_log) > lim[j] + 1;
    }
    edge = __any(edge);
    auto block = [&](auto first_tag, int kb) __attribute__((always_inline)) {
      constexpr bool FIRST = decltype(first_tag)::value;
      const int key0 = (chunk << block_log) + kb;
      f32x4 s[NT][2];
      turn(kf[0]);
      turn(kf[1]);
#pragma unroll
      for (int ks = 0; ks < NS; ks++)
#pragma unroll
        for (int kt = 0; kt < 2; kt++)
#pragma unroll
          for (int j = 0; j < NT; j++)
            s[j][kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kt][ks], qf[j][ks], ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : s[j][kt], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (kb + 32 < a.block) load_k(key0 + 32);
      if (__builtin_expect(edge, 0)) {
#pragma unroll
        for (int j = 0; j < NT; j++) {
          const int past = lim[j] - key0 - 4 * kq;
#pragma unroll
          for (int kt = 0; kt < 2; kt++)
#pragma unroll
            for (int i = 0; i < 4; i++) s[j][kt][i] = 16 * kt + i > past ? -INFINITY : s[j][kt][i];
        }
      }
      u32x4 pb[NT];
      float tmax[NT];
      bool raise = false;
#pragma unroll
      for (int j = 0; j < NT; j++) {
        float x = -INFINITY;
#pragma unroll
        for (int i = 0; i < 8; i += 2) x = fmaxf(fmaxf(x, s[j][i >> 2][i & 3]), s[j][i >> 2][(i & 3) + 1]);
        tmax[j] = fmaf(x, a.c1, bias[j]);
        // an item begins with its own maximum: with the rows' present one the result would depend on which wave was faster
        if (FIRST) m_ref[j] = quad_rows_max(tmax[j]);
        else raise |= tmax[j] > m_ref[j] + kLazy;
      }
      if (!FIRST && __builtin_expect(__any(raise), 0)) {
#pragma unroll
        for (int j = 0; j < NT; j++) {
          const float m_new = fmaxf(m_ref[j], quad_rows_max(tmax[j])), m_use = m_new == -INFINITY ? 0.f : m_new;
          const float corr = __builtin_amdgcn_exp2f(m_ref[j] - m_use);
          m_ref[j] = m_new;
          l[j] *= corr;
#pragma unroll
          for (int e = 0; e < NE; e++)
#pragma unroll
            for (int i = 0; i < 4; i++) acc[j][e][i] *= corr;
        }
      }
#pragma unroll
      for (int j = 0; j < NT; j++) {
        const float off = bias[j] - (m_ref[j] == -INFINITY ? 0.f : m_ref[j]);
        float p[8], sum = 0.f;
#pragma unroll
        for (int i = 0; i < 8; i++) {
          p[i] = __builtin_amdgcn_exp2f(fmaf(s[j][i >> 2][i & 3], a.c1, off));
          sum += p[i];
        }
        l[j] = FIRST ? sum : l[j] + sum;
#pragma unroll
        for (int i = 0; i < 4; i++) pb[j][i] = cvt_bf16x2(p[2 * i], p[2 * i + 1]);
      }
#pragma unroll
      for (int e = 0; e < NE; e++) {
        u32x4 vo;
#pragma unroll
        for (int i = 0; i < 4; i++)
          vo[i] = __builtin_amdgcn_perm(vr[2 * i + 1][e >> 1], vr[2 * i][e >> 1], (e & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
        for (int j = 0; j < NT; j++)
          acc[j][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vo), __builtin_bit_cast(bf16x8, pb[j]), FIRST ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[j][e], 0, 0, 0);
        if (e & 1) __builtin_amdgcn_sched_barrier(0);
      }
      if (kb + 32 < a.block) load_v(key0 + 32);
    };
    block(std::true_type{}, 0);
#pragma clang loop unroll(disable)
    for (int kb = 32; kb < a.block; kb += 32) block(std::false_type{}, kb);
  };
  auto add_up = [&](auto j_tag, int tag_j, float m_j, float l_j, float m_old, float l_old) __attribute__((always_inline)) {
    constexpr int j = decltype(j_tag)::value;
    if (tag_j >= 0) {
      const int row_j = tag_j & 0xff;
      f32x4* po = lo + kq * 256 + row_j;
      f32x4 x[NB];
#pragma unroll
      for (int i = 0; i < NB; i++) x[i] = po[i * 1024];
      // piece i of lane (m, kq): accumulators (4 i + 0..3) % NE, register 4 i / NE
      if (__builtin_expect(__any(m_j > m_old + kLazy), 0)) {
        const float mx = fmaxf(m_old, m_j), f0 = __builtin_amdgcn_exp2f(m_old - mx);
        if (m_j > m_old + kLazy) {
#pragma unroll
          for (int i = 0; i < NB; i++)
#pragma unroll
            for (int e = 0; e < 4; e++) x[i][e] *= f0;
          l_old *= f0;
          m_old = mx;
          if (kq == 0) lm[row_j] = mx;
        }
      }
      const float f = __builtin_amdgcn_exp2f(m_j - (m_old == -INFINITY ? 0.f : m_old));
#pragma unroll
      for (int i = 0; i < NB; i++) {
#pragma unroll
        for (int e = 0; e < 4; e++) x[i][e] = fmaf(acc[j][(4 * i + e) % NE][(4 * i) / NE], f, x[i][e]);
        po[i * 1024] = x[i];
      }
      if (kq == 0) ll[row_j] = fmaf(l_j, f, l_old);
    }
  };

  for (int item = -1;;) {
    int next = 0;
    if (lane == 0) next = __hip_atomic_fetch_add(&ctl[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    next = __builtin_amdgcn_readfirstlane(next);
    const int tag_a = tag[0], tag_b = two ? tag[1] : -1;
    set_up(min(next, n_items - 1));            // behind the last item: that one again, not used
    if (item >= 0) {
#pragma unroll
      for (int j = 0; j < 2; j++) l[j] = quad_rows_sum(l[j]);
      // A tile's sums are added once its tokens' earlier entries are in.  Tile by tile: waiting for both tiles' tokens first takes 3.06 against 2.99 ms at
      // 32k tokens, group of 4, 9 % kept, one head with 8 % 3.77 / 3.66, head dimension 64 1.78 / 1.69; token by token 3.10, 3.77 and 1.76.
      auto add = [&](auto j_tag, int tag_j) __attribute__((always_inline)) {
        constexpr int j = decltype(j_tag)::value;
        const int at = (tag_j & 0xff) / G;
        for (;;) {
          const int done = __hip_atomic_load(&ldone[at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          if (!__any(tag_j >= 0 && done != tag_j >> 8)) break;
          __builtin_amdgcn_s_sleep(1);
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_setprio(2);             // others wait for these sums
        add_up(j_tag, tag_j, m_ref[j], l[j], lm[tag_j & 0xff], ll[tag_j & 0xff]);
        asm volatile("" ::: "memory");             // a wave's LDS operations complete in order
        if (tag_j >= 0) __hip_atomic_store(&ldone[at], (tag_j >> 8) + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __builtin_amdgcn_s_setprio(0);
      };
      add(std::integral_constant<int, 0>{}, tag_a);
      add(std::integral_constant<int, 1>{}, tag_b);
    }
    if (next >= n_items) break;
    turn(qf[0]);
    turn(qf[1]);
    if (two) attend(std::integral_constant<int, 2>{});
    else attend(std::integral_constant<int, 1>{});
    item = next;
  }
  __syncthreads();

  {
    const int orow = tid & 255, t = orow / G;
    if (tid < 512 && t < n_tok) {
      const float lt = ll[orow], inv = lt > 0.f ? 1.f / lt : 0.f;
      uint16_t* op = a.o + b * a.os_b + (int64_t)(r * G + orow % G) * a.os_h + (int64_t)(tok0 + t) * a.os_t;
#pragma unroll
      for (int h = 0; h < 2; h++) {
        const int q4 = (tid >> 8) * 2 + h;
#pragma unroll
        for (int i = 0; i < NB; i += 2) {
          const f32x4 x = lo[(i * 4 + q4) * 256 + orow], y = lo[((i + 1) * 4 + q4) * 256 + orow];
          u32x4 w;
          w[0] = cvt_bf16x2(x[0] * inv, x[1] * inv); w[1] = cvt_bf16x2(x[2] * inv, x[3] * inv);
          w[2] = cvt_bf16x2(y[0] * inv, y[1] * inv); w[3] = cvt_bf16x2(y[2] * inv, y[3] * inv);
          *reinterpret_cast<u32x4*>(op + q4 * (D / 4) + i * 4) = w;
        }
      }
    }
  }
}

// What kCostTiles tiles, spread over the launch, cost in either kernel; the sum decides for the launch (s2_choice).  Tile by tile the launch would
// take both kernels' longest lists one after the other (2000 tokens against a 32k cache 583 -> 817 us).  A workgroup takes one tile, a wave 32 of its
// rows, as in s2_attend_kernel.  There, in units of 0.2 us of half a CU, a chunk that one of the tile's tokens kept costs the workgroup 4 and another 1 for
// each wave that takes part; here an item of 64 keys costs 5.85 of them per workgroup of a whole CU (head dimension 64: 5.15 of its own, shorter unit), and
// of 128 keys 3.9 (4.0) per 64.  An item holds up to 32 / g_q tokens of a chunk, and on average three tenths of the chunks have one that is
// not full.  Fitted to both kernels' times over 94 launches (16k and 32k tokens and 2000 against a 32k cache, groups of 1 to 8, both head dimensions and chunk
// sizes, 2 to 60 % of the chunks kept, queries independent and correlated): the choice takes 0.7 % more time than the faster kernel of each, and
// none of them more than s2_attend_kernel.  The 12 launches of 2000 tokens lie below kMinTiles and are not given the choice.  32k tokens, there -> here: group of 4, 9 % kept 4.50 -> 3.00 ms, 26 % 6.72 -> 6.05 (not taken), 41 % 7.3 -> 8.5 (not
// taken); 9 % with correlated queries 2.44 -> 2.65 (not taken); chunks of 128, 16 % 5.84 -> 3.26; group of 1, 3 % 5.42 -> 2.9, 8 % 7.48 -> 3.66; head
// dimension 64, 9 % 3.06 -> 1.69.
__global__ __launch_bounds__(256) void s2_costs_kernel(S2Args a, float per_item) {
  __shared__ uint32_t all[64], own[4][64];
  __shared__ int sums[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = a.n_tiles * a.hb, at = (int)((int64_t)blockIdx.x * n / kCostTiles) + blockIdx.x % a.hb;
  const int id = at < n ? at : n - 1;
  const int64_t pair = id % a.hb;
  const int tokw = 32 / a.g_q, tok0 = (id / a.hb * 4 + wave) * tokw;
  for (int i = tid; i < 256; i += 256) own[i >> 6][i & 63] = 0u;
  if (tid < 64) all[tid] = 0u;
  if (tid < 2) sums[tid] = 0;
  if (blockIdx.x == 0) a.choice->arrived[tid] = 0;
  __syncthreads();
  const int words = min(tokw, a.n_q - tok0) * a.words;
  const uint32_t* rows = a.mask + (pair * a.n_q + tok0) * a.words;
  int kept = 0, waves = 0;
  for (int i0 = lane; i0 - lane < words; i0 += 8 * 64) {
    uint32_t w[8];
#pragma unroll
    for (int k = 0; k < 8; k++) w[k] = i0 + 64 * k < words ? rows[i0 + 64 * k] : 0u;
#pragma unroll
    for (int k = 0; k < 8; k++) {
      kept += __popc(w[k]);
      if (w[k]) atomicOr(&own[wave][(i0 + 64 * k) % a.words], w[k]);
    }
  }
  __syncthreads();
  const uint32_t mine = own[wave][lane];
  waves = __popc(mine);
  if (mine) atomicOr(&all[lane], mine);
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) { kept += __shfl_xor(kept, o); waves += __shfl_xor(waves, o); }
  if (lane == 0) { atomicAdd(&sums[0], kept); atomicAdd(&sums[1], waves); }
  __syncthreads();
  if (wave > 0) return;
  int chunks = __popc(all[lane]);
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) chunks += __shfl_xor(chunks, o);
  const float items = (float)sums[0] * (float)a.g_q * (1.f / 32.f) + 0.3f * (float)chunks;
  const float more = per_item * items - (4.f * (float)chunks + (float)sums[1]);
  if (lane == 0)
    __hip_atomic_store(&a.choice->costs[blockIdx.x], (uint64_t)a.call << 32 | __float_as_uint(more), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// 64 records: that many calls in flight on a GPU have one each.
constexpr int kChoices = 64;
static __device__ S2Choice choices[kChoices];
static std::atomic<void*> g_choices[64];          // their address, per device ordinal; nullptr = not asked for yet
static std::atomic<uint32_t> g_calls;

void s2_take_choice(S2Args& a) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return;
  void* at = g_choices[dev].load(std::memory_order_acquire);
  if (!at) {
    if (hipGetSymbolAddress(&at, HIP_SYMBOL(choices)) != hipSuccess || !at) {
      (void)hipGetLastError();                    // the launch goes to s2_attend_kernel
      return;
    }
    g_choices[dev].store(at, std::memory_order_release);
  }
  do a.call = g_calls.fetch_add(1, std::memory_order_relaxed) + 1; while (a.call == 0);   // 0: a record that no call had yet
  a.choice = static_cast<S2Choice*>(at) + a.call % kChoices;
}

hipError_t launch_s2_costs(const S2Args& a, int d, hipStream_t st) {
  const float per_item = d == 128 ? (a.block == 64 ? 5.85f : 3.9f) : (a.block == 64 ? 5.15f : 4.f);
  hipLaunchKernelGGL(s2_costs_kernel, dim3(kCostTiles), dim3(256), 0, st, a, per_item);
  return hipGetLastError();
}

template <int D, int G>
static hipError_t launch_t(const S2Args& a, hipStream_t st) {
  auto kern = s2_gather_kernel<D, G>;
  static LdsOptIn opt_in;
  const size_t lds = GatherCfg<D, G>::lds_bytes(a.words);
  if (hipError_t e = allow_dyn_lds((const void*)kern, lds, opt_in); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((a.n_tiles + 1) / 2 * a.hb), dim3(GatherCfg<D, G>::WAVES * 64), lds, st, a);
  return hipGetLastError();
}

hipError_t launch_s2_gather(const S2Args& a, int d, hipStream_t st) {
  switch (a.g_q) {
    case 1: return d == 128 ? launch_t<128, 1>(a, st) : launch_t<64, 1>(a, st);
    case 2: return d == 128 ? launch_t<128, 2>(a, st) : launch_t<64, 2>(a, st);
    case 4: return d == 128 ? launch_t<128, 4>(a, st) : launch_t<64, 4>(a, st);
    default: return d == 128 ? launch_t<128, 8>(a, st) : launch_t<64, 8>(a, st);
  }
}

template <int D> static size_t lds_bytes(int g, int words) {
  return g == 1 ? GatherCfg<D, 1>::lds_bytes(words) : g == 2 ? GatherCfg<D, 2>::lds_bytes(words) : g == 4 ? GatherCfg<D, 4>::lds_bytes(words) : GatherCfg<D, 8>::lds_bytes(words);
}

// Groups of 16: a wave of the other kernel has two tokens, and this one is slower at every density measured (5 to 100 % kept, 0.41 to 0.81 times as
// fast).  The lists' words have to fit beside the sums: up to 576 chunks at a group of 1, 1152 at 2, any number at 4 and 8 (head dimension 128).
bool s2_may_gather(const S2Args& a, int d) {
  const int64_t tiles = (int64_t)a.n_tiles * a.hb * ((a.causal ? a.pos0 + a.n_q / 2 : a.n_kv) / 64);
  return a.g_q <= 8 && a.t_all >= 64 && tiles >= kMinTiles && (d == 128 ? lds_bytes<128>(a.g_q, a.words) : lds_bytes<64>(a.g_q, a.words)) <= 160 * 1024;
}

}  // namespace dash
