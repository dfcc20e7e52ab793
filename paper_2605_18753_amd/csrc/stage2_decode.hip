// Host side of the bf16 decode kernels (decode_body.h), the attention over given lists and the
// dense reference, and the scoring launch of long caches.
#include <math.h>
#include <stdlib.h>

#include <atomic>
#include <chrono>

#include "decode_body.h"

namespace dash {

hipError_t launch_decode_route_m0(const DecArgs& a, int head_dim, unsigned grid, size_t lds, hipStream_t st);
hipError_t launch_decode_route_m1(const DecArgs& a, int head_dim, unsigned grid, size_t lds, hipStream_t st);
hipError_t launch_decode_route_m2(const DecArgs& a, int head_dim, unsigned grid, size_t lds, hipStream_t st);
hipError_t launch_decode_route_m3(const DecArgs& a, int head_dim, unsigned grid, size_t lds, hipStream_t st);
hipError_t launch_decode_route_m4(const DecArgs& a, int head_dim, unsigned grid, size_t lds, hipStream_t st);

// A number for the split flags that no other call of this process uses and that left-over
// memory does not hold: a counter started from the clock, mixed (splitmix64).
static uint64_t next_nonce() {
  static std::atomic<uint64_t> count{(uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() << 20};
  uint64_t z = count.fetch_add(1, std::memory_order_relaxed) * 0x9e3779b97f4a7c15ull + 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  z ^= z >> 31;
  return z ? z : 1;
}

// Scores of all candidate chunks of a pair, 64 chunks per workgroup (a 16-chunk tile per wave).
template <int D, bool WIDE>
__global__ __launch_bounds__(256) void s1_decode_scores_kernel(DecArgs a, float* scores) {
  const S2Args& s = a.s;
  const int pair = blockIdx.x % s.hb, r = pair % s.h_kv, b = pair / s.h_kv;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int len = s.seq_lens ? min(max(s.seq_lens[b], 1), s.n_kv) : s.n_kv;
  const int n_cand = min(max((len - 1) / s.block - a.window, 0), a.t_c);
  const int ct = (blockIdx.x / s.hb) * 4 + wave;
  if (ct * 16 >= n_cand) return;
  DecScore<D, WIDE> sc;
  f32x4 kv[DecScore<D, WIDE>::NS];
  sc.load_tile(a.kbar + (int64_t)pair * a.t_c * D, ct, n_cand, lane, kv);
  sc.load_q(s.q + b * s.qs_b + (int64_t)r * s.g_q * s.qs_h, s.qs_h, s.g_q, lane);
  sc.use_tile(kv, ct, n_cand, s.g_q, a.xscale, lane, scores + (int64_t)pair * s.g_q * a.ld_scores, a.ld_scores);
}

template <int D, int KIND>
static hipError_t launch_attend_t(const DecArgs& a, size_t lds, hipStream_t st) {
  auto kern = s2_decode_kernel<D, KIND, MODE_P2, false>;
  static LdsOptIn opt_in;
  if (hipError_t e = allow_dyn_lds((const void*)kern, lds, opt_in); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(a.n_main), dim3(256), lds, st, a);
  return hipGetLastError();
}

// entries a split's share can hold (host bound of the kernel's split rule)
static int share_cap(const dash_params& p, const Layout& L) {
  int cap = L.t_all;
  if (!L.seq_lens) {
    if (L.splits > 1) cap = (L.t_all + L.splits - 1) / L.splits + 2;      // a share may start and end inside a chunk
  } else {
    const int64_t extra = L.slots - (int64_t)(L.slots / (2 * p.batch) > 1 ? L.slots / (2 * p.batch) : 1) * p.batch;
    if (extra > 0) {
      const int64_t c = ((int64_t)p.batch * L.t_all + extra - 1) / extra + 4;
      cap = c < L.t_all ? (int)c : L.t_all;
    }
    if (cap < (L.t_all + 63) / 64 + 2) cap = (L.t_all + 63) / 64 + 2;
  }
  return cap < L.t_all ? cap : L.t_all;
}

static DecArgs make_dec_args(const dash_params& p, const Layout& L, const void* q, const void* k, const void* v, void* o,
                             const uint32_t* mask, const float* bias, char* ws) {
  DecArgs a{};
  fill_s2_args(a.s, p, L, q, k, v, o, mask, bias);
  a.s.part = reinterpret_cast<float*>(ws + L.off_part);
  a.flags = reinterpret_cast<uint64_t*>(ws + L.off_flags);
  a.splits = L.splits; a.slots = L.slots; a.batch = p.batch;
  a.n_main = L.seq_lens ? p.h_kv * L.slots : p.batch * p.h_kv * L.splits;
  a.nonce = next_nonce();
  a.share_cap = (share_cap(p, L) + 3) & ~3;
  const size_t ring = p.head_dim == 128 ? DecCfg<128>::RING_BYTES : DecCfg<64>::RING_BYTES;
  a.rows_cap = (int)(ring / 4);
  return a;
}

static size_t dec_lds_bytes(const DecArgs& a) { return ((size_t)a.rows_cap + a.share_cap) * 4 + DecCfg<128>::MISC_BYTES; }

hipError_t launch_decode_s2(const dash_params& p, const Layout& L, const void* q, const void* k,
                            const void* v, void* o, const uint32_t* mask, const float* bias,
                            char* ws, bool dense, hipStream_t st) {
  const DecArgs a = make_dec_args(p, L, q, k, v, o, mask, bias, ws);
  const size_t lds = dec_lds_bytes(a);
  if (p.head_dim == 128) return dense ? launch_attend_t<128, DEC_DENSE>(a, lds, st) : launch_attend_t<128, DEC_LISTS>(a, lds, st);
  return dense ? launch_attend_t<64, DEC_DENSE>(a, lds, st) : launch_attend_t<64, DEC_LISTS>(a, lds, st);
}

// Score area (floats) of a decode workgroup that scores by itself: the g_q rows, and the four
// waves' sums over them.
static size_t score_floats(const Layout& L, int rows) { return (size_t)(rows > 4 ? rows : 4) * (((L.t_c + 15) / 16) * 16 + 4); }
constexpr size_t kMaxScoreBytes = 66 * 1024;   // two workgroups per CU with their biases

// Where the scores of a decode step are computed.  In the attention's own workgroups each of a pair's
// splits repeats them: about 16 n_cand clocks per CU (two workgroups reading 512 n_cand bytes of
// summaries each at 64 B/clk) for groups of up to 4 heads, 32 n_cand for larger ones (their
// v_mfma_f32_16x16x4 rate).  A launch of its own costs about 4 us = 10^4 clocks and pays beyond
// that.
// The thresholds are solved in those workgroups too.  That is cheap except for alpha > 2, a bisection of some 25 evaluations
// with a logarithm and an exponential per chunk: there only up to 64 row slots of 64 chunks per CU, beyond
// which one workgroup of 16 waves per pair (dash_stage1_route's kernel, then the attention over its lists) is faster.
// alpha 3, us per step, solved here / in a launch: 16 x 8 pairs of 30000 tokens, group of 4 (64 slots) 47 / 85; 4 x 4 of
// 40000 (128) 60 / 40; 24 x 2 of 20000, group of 16 (256) 97 / 64; 4 x 2 of 65000, group of 8, scores in a launch of their own (256) 84 / 71.
static bool solve_in_place(const dash_params& p, const Layout& L) {
  if (L.pexp >= 1.f) return true;
  int nj = 1;                                  // slots of 64 chunks a wave's registers are laid out for
  while (nj * 64 < L.t_c) nj *= 2;
  return L.g_q * nj * ((int64_t)p.batch * p.h_kv * L.splits > 256 ? 2 : 1) <= 64;
}
static bool score_in_place(const dash_params& p, const Layout& L) {
  return solve_in_place(p, L) && score_floats(L, L.g_q) * 4 <= kMaxScoreBytes && (L.splits == 1 || L.t_c <= (L.g_q > 4 ? 320 : 640));
}
// Score rows of a launch of their own are kept in the workspace, for up to 48 MB of summaries;
// beyond that streaming the summaries takes the time of a routing launch anyway (9 us), and
// dash_stage1_route's kernel followed by the attention over its lists is as fast without the rows.
bool decode_scores_apart(const dash_params& p, const Layout& L) {
  if (p.dtype != DASH_BF16 || p.n_q != 1 || !p.causal || L.t_c <= 0 || !solve_in_place(p, L) || score_in_place(p, L)) return false;
  return (size_t)p.batch * p.h_kv * L.t_c * p.head_dim * 4 < ((size_t)48 << 20);
}

int decode_scores_ld(const Layout& L) { return ((L.t_c + 15) / 16) * 16; }

// Whether the step fits the one-launch kernel with the workspace the caller has (ws_bytes).
bool decode_route_applicable(const dash_params& p, const Layout& L, size_t ws_bytes) {
  if (p.dtype != DASH_BF16) return false;
  return score_in_place(p, L) || (L.dec_scores && ws_bytes >= L.total);
}

hipError_t launch_decode_route(const dash_params& p, const Layout& L, const void* q, const void* k, const void* v, void* o,
                               float* kbar, bool update, const S1Out& out, char* ws, size_t ws_bytes, hipStream_t st) {
  DecArgs a = make_dec_args(p, L, q, k, v, o, nullptr, nullptr, ws);
  a.kbar = kbar;
  a.mask_out = out.mask; a.cnt = out.cnt; a.idx = out.idx; a.bias_out = out.bias; a.tau = out.tau;
  a.t_c = L.t_c; a.window = p.window;
  a.xscale = L.xscale; a.pexp = L.pexp; a.alpha = p.alpha; a.inv_sigma = 1.f / p.sigma;
  const bool apart = L.dec_scores && ws_bytes >= L.total;
  const size_t need = score_floats(L, apart ? 4 : L.g_q);
  if ((size_t)a.rows_cap < need) a.rows_cap = (int)((need + 3) & ~(size_t)3);
  if (apart) {
    float* scores = reinterpret_cast<float*>(ws + L.off_dec_scores);
    a.ld_scores = decode_scores_ld(L);
    const dim3 grid((unsigned)((L.t_c + 63) / 64 * a.s.hb)), blk(256);
    if (p.head_dim == 128) {
      if (L.g_q > 4) hipLaunchKernelGGL((s1_decode_scores_kernel<128, true>), grid, blk, 0, st, a, scores);
      else hipLaunchKernelGGL((s1_decode_scores_kernel<128, false>), grid, blk, 0, st, a, scores);
    } else {
      if (L.g_q > 4) hipLaunchKernelGGL((s1_decode_scores_kernel<64, true>), grid, blk, 0, st, a, scores);
      else hipLaunchKernelGGL((s1_decode_scores_kernel<64, false>), grid, blk, 0, st, a, scores);
    }
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    a.scores = scores;
  }
  // a current token that completes a chunk: one more workgroup per pair summarises it (per-sequence
  // lengths: decided there)
  const bool upd = update && L.t_c > 0 && (L.seq_lens || p.n_kv % p.block_size == 0);
  a.kbar_upd = upd ? kbar : nullptr;
  const unsigned grid = (unsigned)(a.n_main + (upd ? a.s.hb : 0));
  const size_t lds = dec_lds_bytes(a);
  switch (s1_mode(L.pexp)) {
    case MODE_P1: return launch_decode_route_m0(a, p.head_dim, grid, lds, st);
    case MODE_P2: return launch_decode_route_m1(a, p.head_dim, grid, lds, st);
    case MODE_P4: return launch_decode_route_m2(a, p.head_dim, grid, lds, st);
    case MODE_GEN: return launch_decode_route_m3(a, p.head_dim, grid, lds, st);
    default: return launch_decode_route_m4(a, p.head_dim, grid, lds, st);
  }
}

}  // namespace dash
