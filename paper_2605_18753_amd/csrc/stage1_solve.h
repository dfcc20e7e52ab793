// Threshold solver of the Stage-1 kernels that spread a score row over the 64 lanes of a wave
// (stage1.hip; the decode step in stage2_decode.hip).
#pragma once
#include "common.h"
#include "stage1_common.h"

namespace dash {

// Four rows: once a lane's values are summed, it goes on with row l % 4 only, as in stage1_regs.hip (same order of
// additions, same bits as one row at a time).  24 sequences of 32768 tokens, 32 / 2 heads, a step: 66.8 -> 65.5 us.
template <int NJ, int MODE>
__device__ __forceinline__ void solve_four_rows(const float (&v)[4][NJ], int n_cand, float alpha, float p, float (&tau)[4]) {
  const int m = lane_id() & 15;
  auto over_rows = [](float x) {              // the sum of the four DPP rows, in wave_reduce's order
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    const u2 a = __builtin_bit_cast(u2, __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false));
    const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const u2 b = __builtin_bit_cast(u2, __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false));
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
  };
  float ml[4], mx[4];
#pragma unroll
  for (int rb = 0; rb < 4; rb++) {
    ml[rb] = -INFINITY;
#pragma unroll
    for (int j = 0; j < NJ; j++) ml[rb] = fmaxf(ml[rb], v[rb][j]);
    mx[rb] = wave_max(ml[rb]);
  }
  const float top = pick4(mx, m);
  float lo = top - 1.f, hi = top - exp2f(-(alpha - 1.f) * log2f((float)n_cand)), th = lo;
  bool done = false;
  if constexpr (MODE != MODE_BISECT) {
    // warm start on the 64 lane maxima, see solve_rows_regs
    float w[4];
    quad_transpose(ml, w, m);
    for (int it = 0; it < 5; it++) {
      float f[4], g[4];
#pragma unroll
      for (int k = 0; k < 4; k++) {
        pow_terms<MODE>(fmaxf(w[k] - th, 0.f), p, f[k], g[k]);
        asm volatile("" : "+v"(f[k]), "+v"(g[k]));
      }
      const float F = over_rows(add_quads((f[0] + f[1]) + (f[2] + f[3])));
      const float G = over_rows(add_quads((g[0] + g[1]) + (g[2] + g[3])));
      const float st = (F - 1.f) / (p * G);
      th += F > 1.f && G > 0.f ? st : 0.f;
    }
    th = fmaxf(th, lo);
    if (!(th < hi)) th = lo;
  }
  auto spread = [&]() {
    tau[0] = dpp_f<0x00>(th); tau[1] = dpp_f<0x55>(th); tau[2] = dpp_f<0xAA>(th); tau[3] = dpp_f<0xFF>(th);
  };
  spread();
  for (int it = 0; it < 64; it++) {
    float F[4], G[4];
#pragma unroll
    for (int rb = 0; rb < 4; rb++) {
      F[rb] = 0.f; G[rb] = 0.f;
#pragma unroll
      for (int j = 0; j < NJ; j++) {
        float f, g;
        pow_terms<MODE>(fmaxf(v[rb][j] - tau[rb], 0.f), p, f, g);
        F[rb] += f; G[rb] += g;
      }
      asm volatile("" : "+v"(F[rb]), "+v"(G[rb]));         // rounded before the first cross-lane add
    }
    newton_step<MODE>(over_rows(sum4_scatter(F, m)), over_rows(sum4_scatter(G, m)), p, n_cand, th, lo, hi, done);
    spread();
    if (!__any(!done)) break;
  }
}

// Solve RB rows at once (interleaved for ILP): v[rb] holds row rb, lane l chunks l, l+64, ...
// (-inf where absent).  On return v holds the per-head entmax probabilities and tau_out the
// thresholds.
template <int NJ, int RB, int MODE>
__device__ __forceinline__ void solve_rows_regs(float (&v)[RB][NJ], int n_cand, float alpha, float p, float* tau_out /*[RB]*/) {
  if constexpr (RB == 4) {
    float tau[4];
    solve_four_rows<NJ, MODE>(v, n_cand, alpha, p, tau);
#pragma unroll
    for (int rb = 0; rb < 4; rb++) {
#pragma unroll
      for (int j = 0; j < NJ; j++) v[rb][j] = pow_p<MODE>(fmaxf(v[rb][j] - tau[rb], 0.f), p);
      tau_out[rb] = tau[rb];
    }
  } else {
    float mx[RB], lo[RB], hi[RB], tau[RB];
    bool done[RB];
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
      float m = -INFINITY;
#pragma unroll
      for (int j = 0; j < NJ; j++) m = fmaxf(m, v[rb][j]);
      mx[rb] = wave_max(m);
      lo[rb] = mx[rb] - 1.f;
      hi[rb] = mx[rb] - exp2f(-(alpha - 1.f) * log2f((float)n_cand));
      tau[rb] = lo[rb];
      done[rb] = false;
    }
    if constexpr (MODE != MODE_BISECT) {
      // warm start on the 64 lane maxima (a subset: its root and every Newton
      // iterate from the left on it are lower bounds of tau)
      float ml[RB];
#pragma unroll
      for (int rb = 0; rb < RB; rb++) {
        ml[rb] = -INFINITY;
#pragma unroll
        for (int j = 0; j < NJ; j++) ml[rb] = fmaxf(ml[rb], v[rb][j]);
      }
      for (int it = 0; it < 5; it++) {
#pragma unroll
        for (int rb = 0; rb < RB; rb++) {
          float f, g;
          pow_terms<MODE>(fmaxf(ml[rb] - tau[rb], 0.f), p, f, g);
          const float F = wave_sum(f), G = wave_sum(g);
          if (F > 1.f && G > 0.f) tau[rb] += (F - 1.f) / (p * G);
        }
      }
#pragma unroll
      for (int rb = 0; rb < RB; rb++) {
        tau[rb] = fmaxf(tau[rb], lo[rb]);
        if (!(tau[rb] < hi[rb])) tau[rb] = lo[rb];
      }
    }
    for (int it = 0; it < 64; it++) {
      bool all_done = true;
#pragma unroll
      for (int rb = 0; rb < RB; rb++) {
        float F = 0.f, G = 0.f;
#pragma unroll
        for (int j = 0; j < NJ; j++) {
          float f, g;
          pow_terms<MODE>(fmaxf(v[rb][j] - tau[rb], 0.f), p, f, g);
          F += f; G += g;
        }
        F = wave_sum(F);
        G = wave_sum(G);
        // newton_step with its branches: a wave holds whole rows, so all its lanes take the same one.  With newton_step's selects
        // a decode step at alpha 2.5, 25 steps a row, takes 1 to 4 % longer (1000 tokens, 32 / 8 heads 15.8 -> 16.4 us); at alpha 1.25 to
        // 1.7 no difference.  Same bits.
        if (!done[rb]) {
          const float f = F - 1.f;
          if (f == 0.f) {
            done[rb] = true;
          } else {
            if (f > 0.f) lo[rb] = tau[rb]; else hi[rb] = tau[rb];
            const float mid = 0.5f * (lo[rb] + hi[rb]);
            float cand = (MODE == MODE_BISECT || !(G > 0.f)) ? mid : tau[rb] + f / (p * G);
            if (MODE != MODE_BISECT && cand == tau[rb]) {
              done[rb] = true;                       // Newton step below the fp32 spacing of tau
            } else {
              if (!(cand > lo[rb] && cand < hi[rb])) cand = mid;
              if (!(cand > lo[rb] && cand < hi[rb])) {
                done[rb] = true;                     // bracket closed: adjacent floats
                tau[rb] = lo[rb];
              } else {
                if (MODE == MODE_P2 && f > 0.f && cand != mid) {   // see newton_step
                  const float st = cand - tau[rb];
                  if ((float)n_cand * st * st < 4e-8f * G) done[rb] = true;
                }
                tau[rb] = cand;
              }
            }
          }
        }
        all_done = all_done && done[rb];
      }
      if (all_done) break;
    }
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
#pragma unroll
      for (int j = 0; j < NJ; j++) v[rb][j] = pow_p<MODE>(fmaxf(v[rb][j] - tau[rb], 0.f), p);
      tau_out[rb] = tau[rb];
    }
  }
}

}  // namespace dash
