// Routing backward: from the bias gradient dd by chunk to the gradient
// of the entmax scores, and its part of dq; see backward.hip for the chain.
//
// bf16 tensors: a wave owns 16 (token, head) rows: the g_q heads of 16 / g_q tokens, whose candidate sets are the
// same.  It walks the candidates in tiles of 16 chunks, twice: margins u = xscale <q, kbar> - tau,
// weights and slopes, and the row sums of the Jacobian; then dx and dq += dx kbar.  Both products run
// on the fp32 matrix cores in the layouts of f32_tiles.h, the accumulator of the first (lane
// (n, hq): row n, chunks 4 hq .. + 3) being the operand of the second.  The margins of the first walk are
// kept in LDS, lane-private, for rows of up to 256 chunks and computed again beyond.
//
// The gradient is singular at the threshold (1 / w, and for alpha > 2 the slope as well), so a
// chunk next to it magnifies the rounding of its margin.  Margins below kNear therefore come from
// one definition shared with the kernel for fp32 tensors (near_margin: fp32 FMAs in eight
// partial sums), whatever the tiling; about one tile in twenty has one.
//
// What bounds it: L2 reads of the summaries (16 KB per 16 rows and 16 chunks at d = 128), and the
// fp32 matrix rate (its pipe 12 % busy per wave).  Training-shaped workload (4 x 16 heads x 8192 tokens): 1.33 ms with one wave
// per token and fp32 FMAs on 8 lanes per summary row -> 616 us -> 502 with the registers bounded and mask, bias gradient, q and
// tau asked for a tile or a walk ahead (both builds in turn); 24000 tokens, 8 / 2 heads, d 128 and 64: 673 -> 522, 371 -> 259 us;
// 2 x 16 / 4 heads x 3001 tokens of d 64 (at most three tiles a row): 33 us both.
#include <math.h>

#include "backward_args.h"
#include "dash_internal.h"
#include "f32_tiles.h"

namespace dash {

// u^p and p u^(p-1) for u > 0
__device__ __forceinline__ void pow_and_slope(float u, float p, float& w, float& g) {
  if (p == 2.f) { w = u * u; g = 2.f * u; }
  else if (p == 1.f) { w = u; g = 1.f; }
  else { w = __builtin_amdgcn_exp2f(p * __builtin_amdgcn_logf(u)); g = p * w / u; }
}

// sum over the G adjacent lanes of a token; the same value in all of them
template <int G> __device__ __forceinline__ float group_sum(float v) {
  asm volatile("" : "+v"(v));
  if constexpr (G >= 2) v += dpp_f<0xB1>(v);
  if constexpr (G >= 4) v += dpp_f<0x4E>(v);
  if constexpr (G >= 8) v += dpp_f<0x141>(v);
  if constexpr (G >= 16) v += dpp_f<0x140>(v);
  return v;
}

// fp32 tensors: one wave per token, fp32 FMAs, eight lanes per summary row.  The margins are
// formed like the fp32 scores themselves, from fp32 dot products.  These problems are small, and 16
// times as many waves hide their latency better: one head, 1024 tokens, d 64: 5.8 us against
// 7.7 us in 16-row tiles.
template <int D, int G>
__global__ __launch_bounds__(64) void bwd_route_f32_kernel(BwdArgs a) {
  using T = float;
  constexpr int SEG = 64;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  float* qs = reinterpret_cast<float*>(lds);                 // [G][D]
  int* cidx = reinterpret_cast<int*>(qs + G * D);            // [t_c]
  float* dwl = reinterpret_cast<float*>(cidx + a.t_c);       // [t_c]
  float* dxs = dwl + a.t_c;                                  // [G][SEG]

  const int lane = threadIdx.x;
  const int tok = blockIdx.x % a.n_q;
  const int hbi = blockIdx.x / a.n_q;
  const int r = hbi % a.h_kv, b = hbi / a.h_kv;
  const int n_cand = a.causal ? max(tok / a.block - a.window, 0) : a.t_c;
  const int64_t trow = ((int64_t)b * a.h_kv + r) * a.n_q + tok;
  const uint32_t* mrow = a.mask + trow * a.words;
  const float* dbrow = a.dbd + trow * a.t_all;
  const float* kb = a.kbar + ((int64_t)b * a.h_kv + r) * a.t_c * D;

  for (int i = lane; i < G * D; i += 64) {
    const int hh = i / D, d = i % D;
    qs[i] = elem<T>::ld(reinterpret_cast<const T*>(a.q) + b * a.qs_b + (r * G + hh) * a.qs_h + (int64_t)tok * a.qs_t + d);
  }
  // routed candidates, ascending
  int n_r = 0;
  for (int base = 0; base < n_cand; base += 64) {
    const int c = base + lane;
    const bool bit = c < n_cand && ((mrow[c >> 5] >> (c & 31)) & 1u);
    const uint64_t bal = __ballot(bit);
    if (bit) cidx[n_r + __popcll(bal & ((1ull << lane) - 1ull))] = c;
    n_r += __popcll(bal);
  }
  __syncthreads();

  float acc_q[G][2];            // routing part of dq: this lane's d pair (D = 128) or single d (D = 64)
#pragma unroll
  for (int hh = 0; hh < G; hh++) acc_q[hh][0] = acc_q[hh][1] = 0.f;

  if (n_r > 0) {
    float tauh[G];
#pragma unroll
    for (int hh = 0; hh < G; hh++) tauh[hh] = a.tau[((int64_t)b * a.h_q + r * G + hh) * a.n_q + tok];
    float dsum = 0.f;
    for (int e = lane; e < n_r; e += 64) dsum += dbrow[cidx[e]];
    const float dmean = wave_sum(dsum) / (float)n_r;

    // sweep A: scores, weights, slopes; S0 = sum g, S1 = sum g dw_hat per head.
    // Eight lanes share a routed chunk (lane = 8 cs + dp): lane dp reads the dp-th
    // eighth of the summary row, so a wave instruction covers 8 whole rows, and the
    // partial dot products are combined over the 8 lanes by DPP.  Every lane of the
    // group then holds all scores; lane dp keeps the per-head results of the heads
    // hh = dp (mod 8) (slopes to memory, their sums in registers).
    constexpr int DP = D / 8;                      // d range of one lane
    // With few heads the routing part of dq is accumulated in the same sweep:
    // sum_c dx_c kbar_c = sum_c (g_c dw_hat_c) kbar_c - ratio sum_c g_c kbar_c, two sums whose
    // weights are known chunk by chunk, so the summary rows are read once.
    constexpr bool FUSE = 2 * G * DP <= 64;
    const int cs = lane >> 3, dp = lane & 7;
    float s0[G], s1[G];
#pragma unroll
    for (int hh = 0; hh < G; hh++) s0[hh] = s1[hh] = 0.f;
    float a1[FUSE ? G : 1][DP], a2[FUSE ? G : 1][DP];
    if constexpr (FUSE) {
#pragma unroll
      for (int hh = 0; hh < G; hh++)
#pragma unroll
        for (int j = 0; j < DP; j++) a1[hh][j] = a2[hh][j] = 0.f;
    }
    for (int e0 = 0; e0 < n_r; e0 += 8) {
      const int e = e0 + cs;
      const bool live = e < n_r;
      const int c = cidx[live ? e : n_r - 1];
      const float4* krow = reinterpret_cast<const float4*>(kb + (int64_t)c * D + dp * DP);
      float x[G];
#pragma unroll
      for (int hh = 0; hh < G; hh++) x[hh] = 0.f;
      float kvr[DP];
#pragma unroll
      for (int d4 = 0; d4 < DP / 4; d4++) {
        const float4 kv = krow[d4];
        kvr[4 * d4] = kv.x; kvr[4 * d4 + 1] = kv.y; kvr[4 * d4 + 2] = kv.z; kvr[4 * d4 + 3] = kv.w;
#pragma unroll
        for (int hh = 0; hh < G; hh++) {
          const float4 qv = *reinterpret_cast<const float4*>(qs + hh * D + dp * DP + d4 * 4);
          x[hh] = fmaf(qv.x, kv.x, fmaf(qv.y, kv.y, fmaf(qv.z, kv.z, fmaf(qv.w, kv.w, x[hh]))));
        }
      }
      float gd[G], wsum = 0.f;
#pragma unroll
      for (int hh = 0; hh < G; hh++) {
        float xs = x[hh];
        asm volatile("" : "+v"(xs));
        xs += dpp_f<0xB1>(xs);     // lane ^ 1
        xs += dpp_f<0x4E>(xs);     // lane ^ 2
        xs += dpp_f<0x141>(xs);    // the other quad of the 8 lanes
        const float u = xs * a.xscale - tauh[hh];
        float wv = 0.f;
        gd[hh] = 0.f;
        if (u > 0.f) pow_and_slope(u, a.pexp, wv, gd[hh]);
        wsum += wv;
      }
      // dw_hat = dlnw / w / g_q with w = wsum / g_q
      const float dwh = wsum > 0.f ? (dbrow[c] - dmean) / (a.sigma * wsum) : 0.f;
      if (live) {
        if (dp == 0) dwl[e] = dwh;
#pragma unroll
        for (int hh = 0; hh < G; hh++)
          if ((hh & 7) == dp) {
            s0[hh] += gd[hh];
            s1[hh] += gd[hh] * dwh;
            a.dxd[(((int64_t)b * a.h_q + r * G + hh) * a.n_q + tok) * a.t_all + c] = gd[hh];
          }
        if constexpr (FUSE) {
#pragma unroll
          for (int hh = 0; hh < G; hh++) {
            const float w1 = gd[hh] * dwh, w2 = gd[hh];
#pragma unroll
            for (int j = 0; j < DP; j++) {
              a1[hh][j] = fmaf(w1, kvr[j], a1[hh][j]);
              a2[hh][j] = fmaf(w2, kvr[j], a2[hh][j]);
            }
          }
        }
      }
    }
    float ratio[G];
#pragma unroll
    for (int hh = 0; hh < G; hh++) {
      const float t0 = wave_sum(s0[hh]), t1 = wave_sum(s1[hh]);
      ratio[hh] = t0 > 0.f ? t1 / t0 : 0.f;
    }
    if constexpr (FUSE) {
      // dx for the key-owner kernel (each lane turns the slopes it wrote itself into dx)
      for (int e0 = 0; e0 < n_r; e0 += 8) {
        const int e = e0 + cs;
        if (e < n_r) {
          const int c = cidx[e];
          const float dwh = dwl[e];
#pragma unroll
          for (int hh = 0; hh < G; hh++)
            if ((hh & 7) == dp) {
              float* px = a.dxd + (((int64_t)b * a.h_q + r * G + hh) * a.n_q + tok) * a.t_all + c;
              *px = *px * (dwh - ratio[hh]);
            }
        }
      }
      // routing part of dq: combine the two sums, add up the 8 chunk slots (lanes that differ
      // in cs), and hand lane (cs, dp) the d = dp DP + cs DP/8 .. of its output pair
#pragma unroll
      for (int hh = 0; hh < G; hh++) {
        float v0 = 0.f, v1 = 0.f;
#pragma unroll
        for (int j = 0; j < DP; j++) {
          float t = a1[hh][j] - ratio[hh] * a2[hh][j];
          t += __shfl_xor(t, 8);
          t += __shfl_xor(t, 16);
          t += __shfl_xor(t, 32);
          if (D == 128) {
            if ((j >> 1) == cs) { if (j & 1) v1 = t; else v0 = t; }
          } else {
            if (j == cs) v0 = t;
          }
        }
        acc_q[hh][0] = v0;
        acc_q[hh][1] = v1;
      }
    } else
    // sweep B, one segment of SEG routed chunks at a time: dx (each lane turns the slopes
    // it wrote itself into dx), then dq += dx kbar with the lanes over d
    for (int e0 = 0; e0 < n_r; e0 += SEG) {
      __syncthreads();
#pragma unroll
      for (int it = 0; it < SEG / 8; it++) {
        const int j = it * 8 + cs, e = e0 + j;
        if (e < n_r) {
          const int c = cidx[e];
          const float dwh = dwl[e];
#pragma unroll
          for (int hh = 0; hh < G; hh++)
            if ((hh & 7) == dp) {
              float* px = a.dxd + (((int64_t)b * a.h_q + r * G + hh) * a.n_q + tok) * a.t_all + c;
              const float dx = *px * (dwh - ratio[hh]);
              *px = dx;
              dxs[hh * SEG + j] = dx;
            }
        }
      }
      __syncthreads();
      const int cnt = min(SEG, n_r - e0);
      for (int j = 0; j < cnt; j++) {
        const int c = cidx[e0 + j];
        float k0, k1 = 0.f;
        if (D == 128) {
          const float2 kv = *reinterpret_cast<const float2*>(kb + (int64_t)c * D + 2 * lane);
          k0 = kv.x; k1 = kv.y;
        } else {
          k0 = kb[(int64_t)c * D + lane];
        }
#pragma unroll
        for (int hh = 0; hh < G; hh++) {
          const float dx = dxs[hh * SEG + j];
          acc_q[hh][0] = fmaf(dx, k0, acc_q[hh][0]);
          acc_q[hh][1] = fmaf(dx, k1, acc_q[hh][1]);
        }
      }
    }
  }
  // final dq = attention part + routing part; a lane owns the d pair 2 lane .. (D = 128) or the
  // single d = lane (D = 64) in the two-sweep variant, d = 16 dp + 2 cs .. or 8 dp + cs in the fused one
  constexpr bool FUSED = 2 * G * (D / 8) <= 64;
  const int d_own = FUSED ? (D == 128 ? 16 * (lane & 7) + 2 * (lane >> 3) : 8 * (lane & 7) + (lane >> 3))
                          : (D == 128 ? 2 * lane : lane);
#pragma unroll
  for (int hh = 0; hh < G; hh++) {
    const int64_t row = ((int64_t)b * a.h_q + r * G + hh) * a.n_q + tok;
    T* out = reinterpret_cast<T*>(a.dq) + b * a.qs_b + (r * G + hh) * a.qs_h + (int64_t)tok * a.qs_t;
    if (D == 128) {
      const float2 base = *reinterpret_cast<const float2*>(a.dq32 + row * D + d_own);
      const float v0 = fmaf(a.xscale, acc_q[hh][0], base.x), v1 = fmaf(a.xscale, acc_q[hh][1], base.y);
      *reinterpret_cast<float2*>(out + d_own) = make_float2(v0, v1);
    } else {
      elem<T>::st(out + d_own, fmaf(a.xscale, acc_q[hh][0], a.dq32[row * D + d_own]));
    }
  }
}

constexpr float kNear = 1e-4f;

// Margin of one (row, chunk) pair from fp32 FMAs: lane dp = lane % 8 sums the dp-th eighth of the
// head dimension, the partial sums are added pairwise.  q and kbar rows are wave-uniform; all lanes
// get the result.
template <int D> __device__ __forceinline__ float near_margin(const uint16_t* q, const float* kbar, float xscale, float tau, int lane) {
  constexpr int DP = D / 8;
  const int dp = lane & 7;
  float x = 0.f;
#pragma unroll
  for (int d4 = 0; d4 < DP / 4; d4++) {
    const f32x4 kv = *reinterpret_cast<const f32x4*>(kbar + dp * DP + d4 * 4);
    const uint2 w = *reinterpret_cast<const uint2*>(q + dp * DP + d4 * 4);
    x = fmaf(bf16_lo(w.x), kv[0], fmaf(bf16_hi(w.x), kv[1], fmaf(bf16_lo(w.y), kv[2], fmaf(bf16_hi(w.y), kv[3], x))));
  }
  asm volatile("" : "+v"(x));
  x += dpp_f<0xB1>(x);       // lane ^ 1
  x += dpp_f<0x4E>(x);       // lane ^ 2
  x += dpp_f<0x141>(x);      // the other quad of the 8 lanes
  return fmaf(x, xscale, -tau);
}

typedef f32x4 f32x4u __attribute__((aligned(4)));

constexpr int kKeepTiles = 16;   // margin tiles kept in LDS: 1 KB each and wave

// Waves per SIMD that the registers have to leave room for.  Without a bound the accumulators of both products
// are kept twice (109 + 64 registers at d = 128: two waves).  With it, at d = 128: KEEP 126 registers at a group of 1, 122 at
// 16, and 128 with two spilled at 2, 4 and 8 (12 bytes of scratch; with three waves, and none spilled, the whole backward pass takes
// 0.3 % less to 0.4 % more at seven shapes of these groups, and 305 us for 300 at 2 x 16 / 4 heads x 2000 tokens); rows of more
// than 256 chunks 168 with four spilled at a group of 1, six at 2, 4 and 8, none at 16, which is still better than 178 and two
// waves (20001 tokens, 4 heads: 280 us without a bound and the loads ahead, 217 with two waves, 192 with three).  None is spilled
// at d = 64.
constexpr int kRouteWaves = 4, kRouteWavesLong = 3;

template <int D, int G, bool KEEP>
__global__ __launch_bounds__(256, KEEP ? kRouteWaves : kRouteWavesLong) void bwd_route_kernel(BwdArgs a, int n_tiles, int keep_tiles) {
  using C = F32Cfg<D>;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  f32x4* kept = reinterpret_cast<f32x4*>(lds) + (size_t)wave * keep_tiles * 64 + lane;
  const int n = lane & 15, hq = lane >> 4;
  constexpr int TOKT = 16 / G;
  // 4 row tiles per workgroup; the (kv-head, batch) pairs are the fast index; longest rows first
  const int hbi = blockIdx.x % a.hb;
  const int tile = n_tiles - 1 - ((int)(blockIdx.x / a.hb) * 4 + wave);
  if (tile < 0) return;
  const int r = hbi % a.h_kv, b = hbi / a.h_kv;
  const int tok0 = tile * TOKT, tok = min(tok0 + n / G, a.n_q - 1);
  const bool row_ok = tok0 + n / G < a.n_q;
  const int n_cand = a.causal ? max(tok0 / a.block - a.window, 0) : a.t_c;
  const int nct = (n_cand + 15) >> 4;
  const int64_t trow = ((int64_t)b * a.h_kv + r) * a.n_q + tok;
  const int64_t hrow = ((int64_t)b * a.h_q + r * G + n % G) * a.n_q + tok;
  const uint32_t* mrow = a.mask + trow * a.words;
  const float* dbrow = a.dbd + trow * a.t_all;
  float* dxrow = a.dxd + hrow * a.t_all;
  const float* kb = a.kbar + ((int64_t)b * a.h_kv + r) * a.t_c * D;
  const bool wide = a.t_all >= 4;             // a row has four chunks to read at once, at whatever alignment of 4 bytes

  f32x4 dq[C::NS];
#pragma unroll
  for (int i = 0; i < C::NS; i++) dq[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  // this lane's four chunks of a tile: mask bits, and the bias gradient where they are set.  Every lane loads, from
  // inside its row whatever the tile, and one tile ahead: a load under a condition is waited for where it is merged.
  struct Raw { uint32_t word; f32x4 db; };
  auto raw_of = [&](int ct) -> Raw {
    Raw x;
    x.word = mrow[ct >> 1];
    const int c = ct * 16 + 4 * hq;
    if (wide) {
      x.db = *reinterpret_cast<const f32x4u*>(dbrow + min(c, a.t_all - 4));
    } else {
#pragma unroll
      for (int i = 0; i < 4; i++) x.db[i] = dbrow[min(c + i, a.t_all - 1)];
    }
    return x;
  };
  auto bits_in = [&](int ct, const Raw& x) -> uint32_t {
    const uint32_t f = (x.word >> (16 * (ct & 1) + 4 * hq)) & 15u;
    const int left = n_cand - (ct * 16 + 4 * hq);
    return left >= 4 ? f : (left <= 0 ? 0u : f & ((1u << left) - 1u));
  };
  auto db_in = [&](int ct, const Raw& x, uint32_t bits) -> f32x4 {
    f32x4 v = x.db;
    const int ahead = wide ? ct * 16 + 4 * hq - (a.t_all - 4) : 0;           // > 0: read from that many chunks before
    if (ahead & 1 && ahead > 0) v = f32x4{v[1], v[2], v[3], 0.f};
    if (ahead & 2 && ahead > 0) v = f32x4{v[2], v[3], 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; i++) v[i] = ((bits >> i) & 1u) ? v[i] : 0.f;      // not written where the bit is not set
    return v;
  };
  // dx of all candidates, zero where not routed (the summary gradient reads them all)
  auto put_dx = [&](int ct, f32x4 dx) {
    if (!row_ok) return;
    float* p = dxrow + ct * 16 + 4 * hq;
    const int left = n_cand - (ct * 16 + 4 * hq);
    if (left >= 4) {
      *reinterpret_cast<f32x4u*>(p) = dx;
    } else {
#pragma unroll
      for (int i = 0; i < 4; i++)
        if (i < left) p[i] = dx[i];
    }
  };
  // what the second walk starts with arrives during the first
  const uint16_t* qrow = a.q + b * a.qs_b + (int64_t)r * G * a.qs_h;
  uint2 qw[C::NS];
  {
    const uint16_t* qp = qrow + (n % G) * a.qs_h + (int64_t)tok * a.qs_t + 4 * hq;
#pragma unroll
    for (int s = 0; s < C::NS; s++) qw[s] = *reinterpret_cast<const uint2*>(qp + 16 * s);
  }
  const float tau = a.tau[hrow];
  float dsum = 0.f, cnt = 0.f;
  Raw nx = raw_of(0);
  for (int ct = 0; ct < nct; ct++) {
    const Raw x = nx;
    nx = raw_of(ct + 1 < nct ? ct + 1 : 0);
    const uint32_t bits = bits_in(ct, x);
    const f32x4 db = db_in(ct, x, bits);
    dsum += (db[0] + db[1]) + (db[2] + db[3]);
    cnt += (float)__popc(bits);
  }
  dsum = quad_rows_sum(dsum);
  cnt = quad_rows_sum(cnt);
  const float dmean = cnt > 0.f ? dsum / cnt : 0.f;

  if (__any(cnt > 0.f)) {
    f32x4 qf[C::NS];
#pragma unroll
    for (int s = 0; s < C::NS; s++) qf[s] = f32x4{bf16_lo(qw[s].x), bf16_hi(qw[s].x), bf16_lo(qw[s].y), bf16_hi(qw[s].y)};
    auto margins = [&](int ct, uint32_t bits) -> f32x4 {
      f32x4 kf[C::NS];
      load_row<D>(kb + (int64_t)min(ct * 16 + n, n_cand - 1) * D, hq, kf);
      f32x4 u = mma_dot<D>(kf, qf);
#pragma unroll
      for (int i = 0; i < 4; i++) {
        u[i] = fmaf(u[i], a.xscale, -tau);
        uint64_t near = __ballot(((bits >> i) & 1u) && fabsf(u[i]) < kNear);
        while (near) {
          const int l = __builtin_ctzll(near);
          near &= near - 1ull;
          const int row = l & 15, tk = min(tok0 + row / G, a.n_q - 1);
          const float un = near_margin<D>(qrow + (row % G) * a.qs_h + (int64_t)tk * a.qs_t, kb + (int64_t)(ct * 16 + 4 * (l >> 4) + i) * D,
                                          a.xscale, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(tau), l)), lane);
          if (lane == l) u[i] = un;
        }
      }
      return u;
    };
    // slopes g and dw_hat = dlnw / w / g_q (w = wsum / g_q) of this lane's four chunks
    auto terms = [&](const f32x4& um, const f32x4& db, uint32_t bits, f32x4& g, f32x4& dwh) {
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const float u = um[i];
        float w = 0.f, gi = 0.f;
        if (((bits >> i) & 1u) && u > 0.f) pow_and_slope(u, a.pexp, w, gi);
        const float ws = group_sum<G>(w);
        g[i] = gi;
        dwh[i] = ws > 0.f ? (db[i] - dmean) / (a.sigma * ws) : 0.f;
      }
    };
    float s0 = 0.f, s1 = 0.f;
    for (int ct = 0; ct < nct; ct++) {
      const Raw x = nx;
      nx = raw_of(ct + 1 < nct ? ct + 1 : 0);
      const uint32_t bits = bits_in(ct, x);
      if (!__any(bits != 0u)) continue;
      const f32x4 db = db_in(ct, x, bits), u = margins(ct, bits);
      if constexpr (KEEP) kept[ct * 64] = u;
      f32x4 g, dwh;
      terms(u, db, bits, g, dwh);
#pragma unroll
      for (int i = 0; i < 4; i++) { s0 += g[i]; s1 = fmaf(g[i], dwh[i], s1); }
    }
    s0 = quad_rows_sum(s0);
    s1 = quad_rows_sum(s1);
    const float ratio = s0 > 0.f ? s1 / s0 : 0.f;
    for (int ct = 0; ct < nct; ct++) {
      const Raw x = nx;
      nx = raw_of(ct + 1 < nct ? ct + 1 : 0);
      const uint32_t bits = bits_in(ct, x);
      if (!__any(bits != 0u)) { put_dx(ct, f32x4{0.f, 0.f, 0.f, 0.f}); continue; }
      f32x4 kr[4][C::NV];
#pragma unroll
      for (int t = 0; t < 4; t++) load_row2<D>(kb + (int64_t)min(ct * 16 + 4 * hq + t, n_cand - 1) * D, n, kr[t]);
      const f32x4 db = db_in(ct, x, bits);
      f32x4 u, g, dwh, dx;
      if constexpr (KEEP) u = kept[ct * 64]; else u = margins(ct, bits);
      terms(u, db, bits, g, dwh);
#pragma unroll
      for (int i = 0; i < 4; i++) dx[i] = g[i] * (dwh[i] - ratio);
      put_dx(ct, dx);
#pragma unroll
      for (int t = 0; t < 4; t++) mma_outer<D>(kr[t], dx[t], dq);
    }
  }
  else {
    for (int ct = 0; ct < nct; ct++) put_dx(ct, f32x4{0.f, 0.f, 0.f, 0.f});
  }
  // final dq = attention part + routing part
  if (!row_ok) return;
  const float* base = a.dq32 + hrow * D;
  uint16_t* out = a.dq + b * a.qs_b + (r * G + n % G) * a.qs_h + (int64_t)tok * a.qs_t;
#pragma unroll
  for (int nv = 0; nv < C::NV; nv++)
#pragma unroll
    for (int v = 0; v < 4; v++) {
      const int d0 = 64 * nv + 16 * hq + 4 * v;
      const f32x4 bs = *reinterpret_cast<const f32x4*>(base + d0);
      f32x4 y;
#pragma unroll
      for (int e = 0; e < 4; e++) y[e] = fmaf(a.xscale, dq[4 * nv + e][v], bs[e]);
      uint2 w;
      w.x = pack_bf16x2(y[0], y[1]);
      w.y = pack_bf16x2(y[2], y[3]);
      *reinterpret_cast<uint2*>(out + d0) = w;
    }
}

template <int D, int G> static hipError_t launch_route(const BwdArgs& a, hipStream_t st) {
  constexpr int TOKT = 16 / G;
  const int n_tiles = (a.n_q + TOKT - 1) / TOKT;
  const dim3 grid((unsigned)((n_tiles + 3) / 4 * a.hb)), blk(256);
  int max_cand = a.causal ? (a.n_q - 1) / a.block - a.window : a.t_c;
  max_cand = max_cand < 0 ? 0 : (max_cand > a.t_c ? a.t_c : max_cand);
  const int keep = (max_cand + 15) / 16;
  if (keep <= kKeepTiles) {
    auto kern = bwd_route_kernel<D, G, true>;
    const size_t lds = (size_t)4 * keep * 1024;
    static LdsOptIn opt_in;
    if (hipError_t e = allow_dyn_lds((const void*)kern, lds, opt_in); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, blk, lds, st, a, n_tiles, keep);
  } else {
    hipLaunchKernelGGL((bwd_route_kernel<D, G, false>), grid, blk, 0, st, a, n_tiles, 0);
  }
  return hipGetLastError();
}

template <int D, int G> static hipError_t launch_route_f32(const BwdArgs& a, hipStream_t st) {
  const size_t lds = (size_t)G * D * 4 + (size_t)a.t_c * 8 + (size_t)G * 64 * 4 + 64;
  // at most 29 KB of LDS (t_c <= 2048): no opt-in needed
  hipLaunchKernelGGL((bwd_route_f32_kernel<D, G>), dim3((unsigned)((size_t)a.hb * a.n_q)), dim3(64), lds, st, a);
  return hipGetLastError();
}

template <int D> static hipError_t launch_route_g(const BwdArgs& a, bool bf16, hipStream_t st) {
  switch (a.g_q) {
    case 1: return bf16 ? launch_route<D, 1>(a, st) : launch_route_f32<D, 1>(a, st);
    case 2: return bf16 ? launch_route<D, 2>(a, st) : launch_route_f32<D, 2>(a, st);
    case 4: return bf16 ? launch_route<D, 4>(a, st) : launch_route_f32<D, 4>(a, st);
    case 8: return bf16 ? launch_route<D, 8>(a, st) : launch_route_f32<D, 8>(a, st);
    default: return bf16 ? launch_route<D, 16>(a, st) : launch_route_f32<D, 16>(a, st);
  }
}

hipError_t launch_bwd_route(const BwdArgs& a, int head_dim, bool bf16, hipStream_t st) {
  return head_dim == 128 ? launch_route_g<128>(a, bf16, st) : launch_route_g<64>(a, bf16, st);
}

}  // namespace dash
