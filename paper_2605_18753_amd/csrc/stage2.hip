// Stage 2 (bf16 prefill): block-sparse softmax attention over the routed chunks
// with the Stage-1 bias added to the logits (Sec. 3.3 Eq. 6 in the bias form of
// Proposition 1; Alg. 3), and the dense reference attention (Eq. 1) from the
// same template.
//
// Tiling.  A workgroup (4 waves) owns 128 (token, head) rows of one kv-head:
// wave w owns 32 rows = all g_q heads of 32/g_q consecutive tokens.  The
// workgroup walks the union of its tokens' chunk masks in ascending order, written out
// as a list of 64-key tiles first.
// Every 64-key tile of K and V is copied once from global memory straight into
// LDS (buffer_load_dwordx4 ... lds, no staging registers), two stages deep.  A wave
// pipelines its tiles: the first product of tile i runs together with the exponentials of
// tile i - 1, the second product of tile i - 1 together with the row maximum of tile i.  A wave skips
// the MFMA work of a chunk none of its tokens kept; rows of a wave that did not keep a chunk
// get bias -inf for it, which keeps the per-token result exact.
//
// What bounds it.  Dense rows and random data: power.  16k causal tokens, group of 4, take 1.92 ms, 1.15 PFLOP/s, the rate of the
// library's 8192^3 product; the same launch on zeros takes a quarter less, at a clock of 2.1 GHz for 1.65.  Timing copies without
// one part: no direct copies -6.5 %, half of them -2.6, no LDS operand reads -9, no exponentials -6, no row maximum -1, neither copies nor operand
// reads -17.5.  Rows that skip tiles, and launches of one workgroup per CU: the time one wave takes for a tile, 2300
// clocks for 1024 of matrix work (2750 while the list was walked in scalar branches and the chunk was set up behind the barrier:
// 32k prefill 8.36 -> 8.01 ms, 2000 tokens against a 32k cache 695 -> 631 us, 16k with a group of 16 1622 -> 1551, 1000 tokens 37.1 -> 36.2).
// The distances of exponentials and operand reads from their use are worth +-1 %.
// Without the pipeline across tiles (softmax of a tile between its own two products): 8.84 ->
// 8.43 ms at the 32k prefill, 110 -> 104 ms at 128k tokens, 820 -> 735 us for 2000 tokens against a
// 32k cache.
//
// LDS layout.  Tiles are row major ([key][d], no padding: the direct copy writes
// 1 KB contiguous per wave instruction) with the 16-byte chunks of every row
// permuted by an XOR pattern chosen per tensor so that the operand reads below
// are free of bank conflicts; the permutation is applied on the global side
// (which chunk a lane fetches), so it costs nothing.
//
// MFMA formulation (v_mfma_f32_32x32x16_bf16, wave64).  Both products are
// computed transposed so that no register shuffle is needed between them:
//   S^T[key,row]  = K[key,:] . Q[row,:]      A = K tile (LDS), B = Q (registers)
//   O^T[d,row]   += V^T[d,key] . P^T[key,row] A = V^T (LDS, transposing read), B = P
// In the 32x32 accumulator layout lane (n = lane%32, h = lane/32) holds, for
// row n, the 16 keys {8q + 4h + i}: exactly the operand-B slots of lane (n, h)
// once the contraction index of the second product is ordered accordingly.  The
// V^T operand is read from the row-major V tile with ds_read_b64_tr_b16, which
// hands each lane four consecutive keys of one d column.  Row max / row sum are
// in-lane plus one cross-half exchange, and the O rescale is a per-lane scalar.
#include <math.h>
#include <stdlib.h>

#include <type_traits>

#include "common.h"
#include "dash_internal.h"
#include "lds_copy.h"
#include "stage2_args.h"
#include "tile_walk.h"

namespace dash {


constexpr int kMaxTiles = 4096;    // 64-key tiles of a sequence: at most 2048 chunks of 64 or 128

template <int D> struct S2Cfg {
  static constexpr int NCH = D / 8;                       // 16-byte chunks per row
  static constexpr int ROW_BYTES = D * 2;
  static constexpr int TILE_BYTES = 64 * ROW_BYTES;       // one K or V tile
  static constexpr int COPIES = TILE_BYTES / 16 / 256;    // copy instructions per thread, tile and tensor
  static constexpr int ROWS_PER_COPY = 256 / NCH;         // rows one copy instruction of the workgroup covers
  static constexpr int RING_BYTES = 4 * TILE_BYTES;          // the K ring [2] and the V ring [2]
  static constexpr size_t LDS_BYTES = (size_t)RING_BYTES + 5 * 64 * 4 + kMaxTiles * 2;   // ring, chunk bitmaps, list of tiles
};

// Chunk permutations (position of logical 16-byte chunk c of tile row `row`).
// K: the A-operand read has lanes n = 0..15 on 16 consecutive rows at the same
// logical chunk, so those rows must spread over all 16 chunk slots of a 256-byte
// bank window.  V: the transposing read has 16 lanes on 4 consecutive rows x 4
// consecutive chunks, so rows r..r+3 must land in different 64-byte groups.
template <int D> __device__ __forceinline__ int k_swz(int row) {
  return D == 128 ? (row & 15) : ((row >> 1) & 7);
}
template <int D> __device__ __forceinline__ int v_swz(int row) {
  return D == 128 ? ((row & 3) << 2) : (((row >> 1) & 1) << 2);
}

constexpr int kMinPartTiles = 8;   // 64-key tiles a part has at least
constexpr int kMaxParts = 1536;    // records of a launch

// PAIR: eight waves, two groups of four with a ring each, on the same 128 rows: the first walks the first half of the chunk list, the
// second the other, and they add up through LDS.  For launches that leave every CU at most one workgroup (see s2_paired): a
// lone wave per SIMD takes three times a tile's matrix time, so the longest list is what such a launch takes.
// WAVES: per SIMD.  At head dimension 64 three fit with operands of the first product read two steps ahead instead of four (168
// registers, and three spilled that only masked keys, a rising maximum and the end of the walk reload; see launch_s2_t).
template <int D, bool DENSE, bool PAIR, int WAVES = 2>
__global__ __launch_bounds__(PAIR ? 512 : 256, WAVES) void s2_attend_kernel(S2Args a) {
  using C = S2Cfg<D>;
  extern __shared__ __attribute__((aligned(1024))) char lds_all[];
  // PAIR: waves 4 .. 7 are a second group with a ring of its own
  const int grp = PAIR ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8) : 0;
  char* lds = lds_all + grp * C::RING_BYTES;
  uint32_t* wgmask = reinterpret_cast<uint32_t*>(lds_all + (PAIR ? 2 : 1) * C::RING_BYTES);   // [64]
  uint32_t* wvmask = wgmask + 64;                                      // [4][64]
  uint16_t* list = reinterpret_cast<uint16_t*>(wgmask + 5 * 64);       // [kMaxTiles]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) & 3;
  const int n = lane & 31, h = lane >> 5;
  // workgroup id -> (tile, kv-head, batch): consecutive ids walk the (head, batch)
  // pairs so that the 8 XCDs (round-robin dispatch) each see few distinct KV streams
  const int hbi = blockIdx.x % a.hb;
  const int tile = a.n_tiles - 1 - blockIdx.x / a.hb;   // longest rows first
  const int part = blockIdx.y;
  const int r = hbi % a.h_kv, b = hbi / a.h_kv;
  const int tokw = 32 / a.g_q;                          // tokens per wave
  const int tok_w0 = tile * 4 * tokw + wave * tokw;     // first token of this wave
  const int sub_log = a.block >> 7;                     // log2 of the 64-key tiles of a chunk

  // ---- per-row constants ---------------------------------------------------
  const int my_tok = tok_w0 + n / a.g_q;
  const int my_head = r * a.g_q + n % a.g_q;
  const bool row_ok = my_tok < a.n_q;
  const int row_pos = a.pos0 + (row_ok ? my_tok : a.n_q - 1);
  // chunk of the wave's tokens (all tokens of a wave share it)
  const int cw = (a.pos0 + (tok_w0 < a.n_q ? tok_w0 : a.n_q - 1)) / a.block;
  const bool wave_ok = tok_w0 < a.n_q;

  // ---- Q fragments (operand B of S^T = K Q^T) ------------------------------
  bf16x8 qf[D / 16];
  {
    const uint16_t* qp = a.q + b * a.qs_b + my_head * a.qs_h +
                         (int64_t)(row_ok ? my_tok : a.n_q - 1) * a.qs_t + h * 8;
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++) qf[ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 16);
  }

  // ---- chunk bitmaps -------------------------------------------------------
  // Every lane tracks the token of its row: the mask word of the present 32 chunks, where in the compact bias list
  // the token's next bias lies, and that value (prefetched).  The lanes of a token ask for the same address.
  const int64_t trk_base = ((int64_t)b * a.h_kv + r) * a.n_q + min(tok_w0, a.n_q - 1);   // uniform; a lane's row by offset
  const uint32_t* trk_mask = DENSE ? nullptr : a.mask + trk_base * a.words;
  const __amdgpu_buffer_rsrc_t trk_bias = __builtin_amdgcn_make_buffer_rsrc(
      DENSE ? nullptr : const_cast<float*>(a.bias) + trk_base * a.t_all, 0, DENSE ? 0 : max(min(tokw, a.n_q - tok_w0), 0) * a.t_all * 4, 0x00020000);
  auto ask_bias = [&](uint32_t at) -> float { return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(trk_bias, at, 0, 0)); };
  const uint32_t trk_m0 = row_ok ? (uint32_t)(n / a.g_q * a.words) : 0u;
  uint32_t trk_at = row_ok ? (uint32_t)(n / a.g_q * a.t_all) * 4u : ~3u;   // of the next bias, in bytes; past the end for lanes without a token
  uint32_t trk_word = 0;
  float trk_old = 0.f, trk_next = 0.f;
  // The first of them is asked for now, or one nearby: the line comes from another die (a launch behind the routing, which wrote it), and
  // the entry itself is known only with the list.  (757 tokens, 32 / 8 heads of 64, learned summaries,
  // the whole call: 29.5 -> 28.6 us; 1000 tokens of head dimension 128 the same.)
  if constexpr (!DENSE) {
    const uint32_t ahead = PAIR ? (grp * a.t_all >> 1) * 4u : (uint32_t)(part * a.t_all / a.max_parts) * 4u;
    trk_next = ask_bias(row_ok ? trk_at + ahead : ~3u);
  }

  for (int i = tid; i < 5 * 64; i += 256) wgmask[i] = 0u;
  if constexpr (!DENSE && !PAIR) {
    if (a.choice && wave == 0) list[0] = s2_choice(a, lane) > 0;   // one wave asks: what the record says may change between two looks
  }
  __syncthreads();
  if constexpr (!DENSE && !PAIR) {
    if (a.choice && __builtin_amdgcn_readfirstlane((int)list[0])) return;   // left to s2_gather_kernel
  }
  if (DENSE) {
    // every chunk up to the wave's own (causal) / every chunk (non-causal)
    const int last = a.causal ? cw : a.t_all - 1;
    if (wave_ok && grp == 0)
      for (int wi = lane; wi < a.words; wi += 64) {
        const int lo = wi * 32;
        uint32_t m = 0u;
        if (last >= lo) m = (last - lo >= 31) ? 0xffffffffu : ((2u << (last - lo)) - 1u);
        wvmask[wave * 64 + wi] = m;
        if (m) atomicOr(&wgmask[wi], m);
      }
  } else {
    if (wave_ok && grp == 0)
      or_mask_rows(a.mask + (((int64_t)b * a.h_kv + r) * a.n_q + tok_w0) * a.words, min(tokw, a.n_q - tok_w0) * a.words,
                   a.words, wvmask + wave * 64, wgmask, lane);
  }
  __syncthreads();

  // ---- the workgroup's list of 64-key tiles ----------------------------------
  // Entry: tile number (< 4096), bits 12 + w: wave w takes part.  Written once: a walk over the mask words between the tiles is a
  // chain of scalar branches, some 400 clocks of the 2750 that one wave per SIMD took for a tile.
  const int n_chunks = list_tiles<PAIR ? 512 : 256>(wgmask, wvmask, list, sub_log, tid);
  __syncthreads();

  // ---- this workgroup's part of it --------------------------------------------
  int n_parts = 1, first = 0, mine = n_chunks;   // chunks before the part, chunks of the part
  int last_it = n_chunks << sub_log;             // iterations 0 .. last_it: one more than tiles; PAIR: those of the longer half
  if constexpr (PAIR) {
    const ListPart half = list_half(n_chunks, grp, sub_log);
    first = half.first;
    mine = half.chunks;
    last_it = half.last_it;
  } else if (a.max_parts > 1) {
    const int per = max((n_chunks + a.max_parts - 1) / a.max_parts, kMinPartTiles >> sub_log);
    n_parts = max((n_chunks + per - 1) / per, 1);
    if (part >= n_parts) return;
    if (part == 0 && tid == 0) a.part_cnt[blockIdx.x] = n_parts;
    first = part * per;
    mine = min(per, n_chunks - first);
    last_it = mine << sub_log;
  }
  const int n_it = mine << sub_log;              // the part's tiles
  list += first << sub_log;
  auto entry = [&](int i) -> int {               // 0 where there is none
    const int at = walk_index(i, n_it);
    const int e = list[max(at, 0)];
    return at < 0 ? 0 : e;
  };
  int e_cur = __builtin_amdgcn_readfirstlane(entry(0)), e_next = __builtin_amdgcn_readfirstlane(entry(1)), e_ahead = 0;
  if (!DENSE) {
    const int u0 = (e_cur & 0xfff) >> sub_log;
    if (first > 0 && n_it > 0 && row_ok) {       // the token's entries before the part's first chunk
      for (int wi = 0; wi < u0 >> 5; wi++) trk_at += 4 * __popc(trk_mask[trk_m0 + wi]);
      trk_at += 4 * __popc(trk_mask[trk_m0 + (u0 >> 5)] & ((1u << (u0 & 31)) - 1u));
    }
    trk_word = trk_mask[trk_m0 + (u0 >> 5)];
    asm volatile("" : "+v"(trk_next));
    if (first > 0) trk_next = ask_bias(trk_at);
  }

  // ---- global -> LDS tile copies -------------------------------------------
  // Copy instruction i of wave w fills the 1 KB LDS segment (4i + w): slot
  // s = (4i + w) * 64 + lane, tile row s / NCH, chunk position s % NCH, which
  // receives logical chunk pos ^ swz(row) of that row.  The swizzle depends only
  // on (w, lane), so each thread keeps one byte offset per tensor; the tile and
  // instruction offsets are scalar (buffer addressing: resource + lane offset +
  // scalar offset).  The resource ends with the last key, so the rows a ragged
  // last tile has beyond n_kv read as zeros instead of touching memory.
  const u32x4 k_rs = make_rsrc(a.k + b * a.ks_b + r * a.ks_h, (((int64_t)a.n_kv - 1) * a.ks_t + D) * 2);
  const u32x4 v_rs = make_rsrc(a.v + b * a.vs_b + r * a.vs_h, (((int64_t)a.n_kv - 1) * a.vs_t + D) * 2);
  const uint32_t lds0 = lds_addr_of(lds);
  const int c_row = (wave * 64 + lane) / C::NCH, c_pos = lane % C::NCH;
  const uint32_t k_off = (uint32_t)(c_row * (int)a.ks_t * 2 + ((c_pos ^ k_swz<D>(c_row)) << 4));
  const uint32_t v_off = (uint32_t)(c_row * (int)a.vs_t * 2 + ((c_pos ^ v_swz<D>(c_row)) << 4));
  const uint32_t k_step = (uint32_t)(C::ROWS_PER_COPY * (int)a.ks_t * 2);
  const uint32_t v_step = (uint32_t)(C::ROWS_PER_COPY * (int)a.vs_t * 2);
  const uint32_t k_tile = (uint32_t)a.ks_t * 128u, v_tile = (uint32_t)a.vs_t * 128u;   // bytes from tile to tile
  uint32_t cp_k = 0, cp_v = 0;   // scalar byte offsets of the K and V tiles being copied
  auto copy_k = [&](int c, int slot) {
    copy16_to_lds(k_rs, lds0 + slot * C::TILE_BYTES + wave * 1024 + c * 4096, k_off, cp_k + c * k_step);
  };
  auto copy_v = [&](int c, int slot) {
    copy16_to_lds(v_rs, lds0 + (2 + slot) * C::TILE_BYTES + wave * 1024 + c * 4096, v_off, cp_v + c * v_step);
  };

  // ---- operand read addresses (in LDS, of slot 0) ------------------------------
  // K, A operand of S^T: lane (n, h) reads logical chunk 2 ks + h of rows n, 32 + n
  uint32_t k_rd[D / 16];
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++)
    k_rd[ks] = lds0 + (uint32_t)(n * C::ROW_BYTES + (((2 * ks + h) ^ k_swz<D>(n)) << 4));
  // V, A operand of O^T (transposing read): lanes 16 g .. 16 g + 15 serve d
  // columns 16 (g & 1) .. + 15 of a d-tile and contraction half h = g >> 1; lane
  // s of the group points at key row 4 h + s / 4, d offset 16 (g & 1) + 4 (s % 4)
  // of d-tile t, which the row's swizzle moved to 64-byte group t ^ swz(row).
  const int s16 = lane & 15, a16 = (lane >> 4) & 1;
  uint32_t v_rd[D / 32];
#pragma unroll
  for (int t = 0; t < D / 32; t++)
    v_rd[t] = lds0 + (uint32_t)((4 * h + (s16 >> 2)) * C::ROW_BYTES +
                                ((((4 * t) ^ v_swz<D>(s16 >> 2)) + 2 * a16 + ((s16 & 3) >> 1)) << 4) + ((s16 & 1) << 3));

  // ---- online-softmax state (base-2 logits) -------------------------------
  float m_run = -INFINITY, l_run = 0.f;
  constexpr int NDT = D / 32;
  f32x16 oacc[NDT];
#pragma unroll
  for (int dt = 0; dt < NDT; dt++)
#pragma unroll
    for (int j = 0; j < 16; j++) oacc[dt][j] = 0.f;

  float bias_row = 0.f;   // bias * log2e of this lane's row for the current chunk
  auto begin_chunk = [&](int u) {
    // the bias of chunk u, which one of the wave's tokens kept, for this lane's row
    if (DENSE || (a.causal && u == cw)) { bias_row = 0.f; return; }
    const bool bit = row_ok && ((trk_word >> (u & 31)) & 1u);
    const float next = trk_old + trk_next;   // one of them is 0
    bias_row = bit ? next * kLog2e : -INFINITY;
    trk_old = bit ? 0.f : next;
    trk_at += bit ? 4u : 0u;
    // One load for every lane, and none that merges values behind it: where only some lanes load, the others' values are
    // merged right behind the load, and the wave waits for memory here instead of at the next chunk (32k prefill 8.64 ->
    // 8.24 ms, 2000 tokens against a 32k cache 735 -> 674 us, 16k with a group of 16 1.62 -> 1.54 ms).  Lanes whose token did not
    // keep the chunk read past the end of the resource, which touches no memory, and keep their value: reading it again took
    // a cache line of every token for each chunk (128k tokens at alpha 2, chunks of 64, 32 / 8 heads: 55 -> 43 to 50 ms, 8 / 2
    // heads 13.3 -> 12.5; chunks of 128 82 -> 79; 32k and 64k tokens the same to 5 % less).
    trk_next = ask_bias(bit ? trk_at : ~3u);
  };

  // ---- the tile pipeline -----------------------------------------------------
  // Iteration i forms S^T of tile i and O^T += V^T P^T of tile i - 1: the exponentials of tile
  // i - 1 run behind the MFMAs of the first product, the row maximum of tile i behind those of the
  // second, so that a wave has matrix work to issue while its vector work completes.  The source is
  // written slot by slot (one MFMA per slot, its operand reads a few slots ahead, a share of the vector work
  // behind it) and the scheduler may not move code across slots.
  //
  // LDS: K ring [2] then V ring [2]; tile i lives in slot i & 1 of both, V one iteration behind K.  At
  // the top of iteration i a wave waits for its own copies (K of tile i, V of tile i - 1), the barrier
  // makes everybody's visible and retires the reads of iteration i - 1 (K of tile i - 1, V of
  // tile i - 2), whose slots the copies of this iteration (K of tile i + 1, V of tile i) overwrite; those are
  // issued one at a time between the MFMAs: a burst right after the barrier would queue all waves
  // behind the 64 B/clk global -> LDS path.
  //
  // Whatever needs no tile stands before the barrier: the chunk's bias, the reference maximum.
  // the loads of Q, issued before those of the masks, must be complete (and known to be) before the tile
  // loop: a wait for them inside the loop would also wait for the tile copies in flight
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) asm volatile("" : "+v"(qf[ks]));
  if (n_it > 0) {
    cp_k = (uint32_t)(e_cur & 0xfff) * k_tile;
#pragma unroll
    for (int c = 0; c < C::COPIES; c++) copy_k(c, 0);
  }
  int pend = 0;                      // a tile whose S^T waits for its softmax and second product
  float bias_old = 0.f, tmax_old = 0.f;
  auto iteration = [&](auto p_tag, int it, f32x16 (&s)[2], f32x16 (&so)[2]) __attribute__((always_inline)) {
    constexpr int P = decltype(p_tag)::value;
    constexpr int NS = D / 8;                                  // MFMAs per product and tile
    constexpr int KAHEAD = WAVES == 3 ? 2 : 4, VAHEAD = 2;
    constexpr int EQ = 12, E0 = 2;                             // exponential pairs before the second product, and before the first MFMA
    const bool cur = it < n_it;
    const int t_cur = e_cur & 0xfff, t_next = e_next & 0xfff;
    const int on = (e_cur >> (12 + wave)) & ((it - n_it) >> 31) & 1;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (!DENSE) {
      const int u = t_cur >> sub_log, un = t_next >> sub_log;
      if (on && (t_cur & sub_log) == 0) begin_chunk(u);
      if ((un ^ u) >> 5) trk_word = trk_mask[trk_m0 + (un >> 5)];   // arrives with the next tile's copies
    }
    // Lazy rescaling: the reference max m_run of a row is only raised when the tile's max
    // exceeds it by more than 2^kLazy; until then p = 2^(t - m_run) may reach 2^kLazy, which fp32 / bf16
    // hold without loss, and the final division by the row sum is unaffected.
    if (pend && __builtin_expect(__any(tmax_old > m_run + kLazy), 0)) {
      const float m_new = fmaxf(m_run, fmaxf(tmax_old, __shfl_xor(tmax_old, 32)));
      const float m_use = m_new == -INFINITY ? 0.f : m_new;
      const float corr = __builtin_amdgcn_exp2f(m_run - m_use);   // m_run = -inf -> 0
      m_run = m_new;
      l_run *= corr;
#pragma unroll
      for (int dt = 0; dt < NDT; dt++)
#pragma unroll
        for (int j = 0; j < 16; j++) oacc[dt][j] *= corr;
    }
    const float off = bias_old - (m_run == -INFINITY ? 0.f : m_run);
    cp_v = (uint32_t)t_cur * v_tile;                           // V of tile i
    cp_k = (uint32_t)t_next * k_tile;                          // K of tile i + 1
    asm volatile("s_barrier" ::: "memory");
    e_ahead = entry(it + 2);
    auto k_read = [&](int i) -> bf16x8 {   // slot i: d slice i / 2, key half i % 2
      return lds_read_b128(k_rd[i >> 1] + (uint32_t)(P * C::TILE_BYTES + (i & 1) * 32 * C::ROW_BYTES));
    };
    auto v_read = [&](int i) -> bf16x8 {   // slot i: contraction step g = i / NDT, d-tile t = i % NDT
      const uint32_t at = v_rd[i % NDT] + (uint32_t)((2 + (P ^ 1)) * C::TILE_BYTES + 16 * (i / NDT) * C::ROW_BYTES);
      return lds_read_tr_pair(at, at + 8 * C::ROW_BYTES);
    };
    u32x4 pb[4];
    float l_tile = 0.f;   // summed by the tile: one chain over all keys of a long row loses digits
    // exponential pair k of tile i - 1: P^T slots 2 (k % 4), + 1 of contraction step g = k / 4
    auto e_pair = [&](int k) {
      const int g = k >> 2, kt = g >> 1, j = 8 * (g & 1) + 2 * (k & 3);
      const float p0 = __builtin_amdgcn_exp2f(fmaf(so[kt][j], a.c1, off));
      const float p1 = __builtin_amdgcn_exp2f(fmaf(so[kt][j + 1], a.c1, off));
      l_tile += p0 + p1;
      const bf16x2 w = {(__bf16)p0, (__bf16)p1};
      uint32_t x = __builtin_bit_cast(uint32_t, w);
      asm volatile("" : "+v"(l_tile), "+v"(x));   // keeps the row sum and the packing in their slot
      pb[g][k & 3] = x;
    };
    // copy instruction c of the iteration: K of tile i + 1, then V of tile i
    auto copies = [&](int c) {
      if (c < C::COPIES) copy_k(c, P ^ 1);                     // behind the last tile: that tile again, into a slot nobody reads
      else if (c < 2 * C::COPIES) copy_v(c - C::COPIES, P);
    };
    bf16x8 vf[NS];
    auto first_product = [&](auto e_tag) {
      constexpr bool EXPS = decltype(e_tag)::value;
      bf16x8 kf[NS];
#pragma unroll
      for (int i = 0; i < KAHEAD; i++) kf[i] = k_read(i);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (EXPS) {
#pragma unroll
        for (int k = 0; k < E0; k++) e_pair(k);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 0; i < NS; i++) {
        if (i + KAHEAD < NS) kf[i + KAHEAD] = k_read(i + KAHEAD);
        if ((i & 1) == 0) copies(i >> 1);
        const int ks = i >> 1, kt = i & 1;
        if (ks == 0) {
          const f32x16 z = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i], qf[ks], z, 0, 0, 0);
        } else {
          s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i], qf[ks], s[kt], 0, 0, 0);
        }
        if constexpr (EXPS) {
#pragma unroll
          for (int k = E0 + i * (EQ - E0) / NS; k < E0 + (i + 1) * (EQ - E0) / NS; k++) e_pair(k);
          if (i >= NS - VAHEAD) vf[i - (NS - VAHEAD)] = v_read(i - (NS - VAHEAD));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // key kpos0 + 4 h + c (c = the compile-time part of the key index of an accumulator
    // register) is dead if it lies after the row's position in the diagonal chunk or past the
    // end of the sequence, i.e. if c > lim
    auto mask_keys = [&]() {
      const int kpos0 = t_cur * 64;
      const bool diag = a.causal && (t_cur >> sub_log) == cw;
      if (__builtin_expect(diag || kpos0 + 64 > a.n_kv, 0)) {
        const int k0 = kpos0 + 4 * h;
        int lim = min(diag ? row_pos - k0 : 0x7fffffff, a.n_kv - 1 - k0);
        asm volatile("" : "+v"(lim));   // keep the per-register comparisons against immediates
#pragma unroll
        for (int kt = 0; kt < 2; kt++)
#pragma unroll
          for (int j = 0; j < 16; j++) {
            const int c = kt * 32 + (j >> 2) * 8 + (j & 3);
            s[kt][j] = c > lim ? -INFINITY : s[kt][j];
          }
      }
    };
    float mloc = -INFINITY;
    auto max_quad = [&](int q) {   // four of the tile's 32 scores per lane
      const int kt = q >> 2, j = 4 * (q & 3);
      mloc = fmaxf(fmaxf(mloc, s[kt][j]), s[kt][j + 1]);
      mloc = fmaxf(fmaxf(mloc, s[kt][j + 2]), s[kt][j + 3]);
    };
    auto second_product = [&]() {
#pragma unroll
      for (int i = 0; i < NS; i++) {
        if (i + VAHEAD < NS) vf[i + VAHEAD] = v_read(i + VAHEAD);
        const int g = i / NDT, t = i % NDT;
        oacc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[i], __builtin_bit_cast(bf16x8, pb[g]), oacc[t], 0, 0, 0);
        // the remaining pairs belong to the last contraction step
        if (EQ + i < 16) e_pair(EQ + i);
        if constexpr (NS == 16) { if (i >= 4 && i < 12) max_quad(i - 4); }
        else if (i >= 4) { max_quad(2 * (i - 4)); max_quad(2 * (i - 4) + 1); }
        __builtin_amdgcn_sched_barrier(0);
      }
      l_run += l_tile;
    };
    if (on) {
      if (pend) first_product(std::true_type{});
      else first_product(std::false_type{});
      mask_keys();
    } else {
      asm volatile("" : "=v"(s[0]), "=v"(s[1]));               // nobody reads them
      if (cur) {
#pragma unroll
        for (int c = 0; c < 2 * C::COPIES; c++) copies(c);
      }
      if (pend) {
#pragma unroll
        for (int i = 0; i < VAHEAD; i++) vf[i] = v_read(i);
#pragma unroll
        for (int k = 0; k < EQ; k++) e_pair(k);
      }
    }
    // The branches rejoin around the second product, and two conditions stand for an else: otherwise the compiler keeps two
    // sets of accumulators and copies one to the other.
    if (pend) {
      __builtin_amdgcn_sched_barrier(0);
      second_product();
    }
    if (!pend && on) {
#pragma unroll
      for (int q = 0; q < 8; q++) max_quad(q);
    }
    // this lane half's max of the base-2 logits s c1 + bias (c1 > 0)
    tmax_old = fmaf(mloc, a.c1, bias_row);
    bias_old = bias_row;
    pend = on;
    e_cur = e_next;
    e_next = __builtin_amdgcn_readfirstlane(e_ahead);
  };
  if (last_it > 0) {
    f32x16 sa[2], sb[2];
    for (int it = 0;;) {
      iteration(std::integral_constant<int, 0>{}, it, sa, sb);
      if (++it > last_it) break;
      iteration(std::integral_constant<int, 1>{}, it, sb, sa);
      if (++it > last_it) break;
    }
  }

  // ---- finalise ------------------------------------------------------------
  const float l_tot = l_run + __shfl_xor(l_run, 32);
  if (n_parts > 1) {
    // record of the part: O^T unnormalised as [d / 4][row][4], running max and sum per row
    const int64_t rec = (int64_t)blockIdx.x * a.max_parts + part;
    const int row = wave * 32 + n;
    f32x4* po = reinterpret_cast<f32x4*>(a.part_o) + rec * (D / 4) * 128 + row;
#pragma unroll
    for (int t = 0; t < NDT; t++)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++)
        po[(t * 8 + q4 * 2 + h) * 128] = f32x4{oacc[t][q4 * 4], oacc[t][q4 * 4 + 1], oacc[t][q4 * 4 + 2], oacc[t][q4 * 4 + 3]};
    if (h == 0) reinterpret_cast<float2*>(a.part_ml)[rec * 128 + row] = make_float2(m_run, l_tot);
    return;
  }
  auto put_tiles = [&](int t0, int t1, float inv) {
    if (!row_ok) return;
    uint16_t* op = a.o + b * a.os_b + my_head * a.os_h + (int64_t)my_tok * a.os_t;
#pragma unroll
    for (int t = t0; t < t1; t++)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        // accumulator t, registers 4 q4 .. + 3: O^T rows 8 q4 + 4 h + i of d-tile t
        const int m0 = q4 * 8 + h * 4;
        uint2 w;
        w.x = cvt_bf16x2(oacc[t][q4 * 4 + 0] * inv, oacc[t][q4 * 4 + 1] * inv);
        w.y = cvt_bf16x2(oacc[t][q4 * 4 + 2] * inv, oacc[t][q4 * 4 + 3] * inv);
        *reinterpret_cast<uint2*>(op + t * 32 + m0) = w;
      }
  };
  if constexpr (PAIR) {
    // The groups add up through LDS: each hands the other half of its d-tiles, as [d / 4][row][4], and its rows' maxima
    // and sums, where its ring was, and writes the other half.
    constexpr int H = NDT / 2;
    const int row = wave * 32 + n;
    __syncthreads();                                           // nobody reads the tiles any more
    auto exchange = [&](auto g_tag) {
      constexpr int G = decltype(g_tag)::value, MINE = G * H, GIVE = (G ^ 1) * H;
      f32x4* xo = reinterpret_cast<f32x4*>(lds) + row;
#pragma unroll
      for (int t = 0; t < H; t++)
#pragma unroll
        for (int q4 = 0; q4 < 4; q4++)
          xo[(t * 8 + q4 * 2 + h) * 128] = f32x4{oacc[GIVE + t][q4 * 4], oacc[GIVE + t][q4 * 4 + 1], oacc[GIVE + t][q4 * 4 + 2], oacc[GIVE + t][q4 * 4 + 3]};
      if (h == 0) reinterpret_cast<float2*>(lds + 3 * C::TILE_BYTES)[row] = make_float2(m_run, l_tot);
      __syncthreads();
      const char* other = lds_all + (G ^ 1) * C::RING_BYTES;
      const float2 ml = reinterpret_cast<const float2*>(other + 3 * C::TILE_BYTES)[row];
      const float M = fmaxf(m_run, ml.x), m_use = M == -INFINITY ? 0.f : M;
      const float w0 = __builtin_amdgcn_exp2f(m_run - m_use), w1 = __builtin_amdgcn_exp2f(ml.x - m_use);
      const float den = fmaf(w0, l_tot, w1 * ml.y);
      const f32x4* xi = reinterpret_cast<const f32x4*>(other) + row;
#pragma unroll
      for (int t = 0; t < H; t++)
#pragma unroll
        for (int q4 = 0; q4 < 4; q4++) {
          const f32x4 x = xi[(t * 8 + q4 * 2 + h) * 128];
#pragma unroll
          for (int e = 0; e < 4; e++) oacc[MINE + t][q4 * 4 + e] = fmaf(w0, oacc[MINE + t][q4 * 4 + e], w1 * x[e]);
        }
      put_tiles(MINE, MINE + H, den > 0.f ? 1.f / den : 0.f);
    };
    if (grp == 0) exchange(std::integral_constant<int, 0>{});
    else exchange(std::integral_constant<int, 1>{});
    return;
  }
  put_tiles(0, NDT, l_tot > 0.f ? 1.f / l_tot : 0.f);
}

// Adds the parts of the tiles that have several: o = sum_p 2^(m_p - M) O_p / sum_p 2^(m_p - M) l_p.
// A workgroup merges 16 rows of a tile; threads 16 i .. + 15 hold 4 consecutive d of them.
template <int D>
__global__ __launch_bounds__(256) void s2_merge_kernel(S2Args a) {
  const int id = blockIdx.x >> 3, n_parts = a.part_cnt[id];
  if (n_parts <= 1) return;
  const int hbi = id % a.hb, tile = a.n_tiles - 1 - id / a.hb;
  const int r = hbi % a.h_kv, b = hbi / a.h_kv;
  const int row = (blockIdx.x & 7) * 16 + (threadIdx.x & 15);
  const int tok = tile * (128 / a.g_q) + row / a.g_q;
  if (tok >= a.n_q) return;
  const int64_t rec = (int64_t)id * a.max_parts;
  const float2* ml = reinterpret_cast<const float2*>(a.part_ml) + rec * 128 + row;
  float M = -INFINITY, den = 0.f;
  for (int p = 0; p < n_parts; p++) M = fmaxf(M, ml[p * 128].x);
  const float m_use = M == -INFINITY ? 0.f : M;
  for (int p = 0; p < n_parts; p++) den = fmaf(__builtin_amdgcn_exp2f(ml[p * 128].x - m_use), ml[p * 128].y, den);
  const float inv = den > 0.f ? 1.f / den : 0.f;
  constexpr int NG = D / 64;                  // groups of 4 d per thread
  const f32x4* po = reinterpret_cast<const f32x4*>(a.part_o) + (rec * (D / 4) + (threadIdx.x >> 4)) * 128 + row;
  f32x4 o[NG];
#pragma unroll
  for (int i = 0; i < NG; i++) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int p = 0; p < n_parts; p++) {
    const float w = __builtin_amdgcn_exp2f(ml[p * 128].x - m_use);
#pragma unroll
    for (int i = 0; i < NG; i++) {
      const f32x4 x = po[((int64_t)p * (D / 4) + i * 16) * 128];
#pragma unroll
      for (int e = 0; e < 4; e++) o[i][e] = fmaf(w, x[e], o[i][e]);
    }
  }
  uint16_t* op = a.o + b * a.os_b + (int64_t)(r * a.g_q + row % a.g_q) * a.os_h + (int64_t)tok * a.os_t + (threadIdx.x >> 4) * 4;
#pragma unroll
  for (int i = 0; i < NG; i++) {
    uint2 w;
    w.x = cvt_bf16x2(o[i][0] * inv, o[i][1] * inv);
    w.y = cvt_bf16x2(o[i][2] * inv, o[i][3] * inv);
    *reinterpret_cast<uint2*>(op + i * 64) = w;
  }
}

template <int D, bool DENSE>
static hipError_t launch_s2_t(const S2Args& a, bool pair, hipStream_t st) {
  using C = S2Cfg<D>;
  if (pair) {
    auto kern = s2_attend_kernel<D, DENSE, true>;
    static LdsOptIn opt_in;
    constexpr size_t lds = C::LDS_BYTES + C::RING_BYTES;
    if (hipError_t e = allow_dyn_lds((const void*)kern, lds, opt_in); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(a.n_tiles * a.hb), dim3(512), lds, st, a);
    return hipGetLastError();
  }
  if (!DENSE && a.choice)
    if (hipError_t e = launch_s2_costs(a, D, st); e != hipSuccess) return e;
  auto kern = s2_attend_kernel<D, DENSE, false>;
  // Head dimension 64: three workgroups per CU where there are more of them than that holds.  Stage 2 alone, two -> three: 16 / 4 heads x 8000
  // tokens (1000 workgroups) 199 -> 172 us, 32 / 8 heads x 16k, queries correlated, 1305 -> 1190, x 32k 5004 -> 4707, 32 / 2 x 16k 1078 -> 970; with fewer
  // the shorter read-ahead is a loss: 512 workgroups 73.5 -> 75.7 us, 528 41.2 -> 42.3, 752 53.7 -> 54.8.
  if constexpr (D == 64) {
    static_assert(C::LDS_BYTES <= 48 * 1024, "both kernels would need their own record of the opt-in");
    if ((int64_t)a.n_tiles * a.hb * a.max_parts > 768) kern = s2_attend_kernel<D, DENSE, false, 3>;
  }
  static LdsOptIn opt_in;
  if (hipError_t e = allow_dyn_lds((const void*)kern, C::LDS_BYTES, opt_in); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(a.n_tiles * a.hb, a.max_parts), dim3(256), C::LDS_BYTES, st, a);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && !DENSE && a.choice) e = launch_s2_gather(a, D, st);
  if (e != hipSuccess || a.max_parts == 1) return e;
  hipLaunchKernelGGL(s2_merge_kernel<D>, dim3(a.n_tiles * a.hb * 8), dim3(256), 0, st, a);
  return hipGetLastError();
}

static int64_t s2_most_records(const dash_params& p, const Layout& L);
static int s2_tiles(const dash_params& p, const Layout& L) { return (p.n_q + 128 / L.g_q - 1) / (128 / L.g_q); }

// Whether a launch that is not cut walks each list with two groups of waves.  It takes as long as the longest half, and a CU has room
// for one such workgroup: no more than 256 of them.  Of up to four tiles the halves gain what the exchange costs (whole forward,
// one group -> two, 32 / 8 heads: 128 tokens 20.7 -> 21.2 us, 192 25.0 -> 25.8, 256 28.2 -> 28.3; 257 29.4 -> 28.5, 500 37.1 -> 33.8,
// 1000 45.9 -> 41.7; 16 heads over one x 2048 66.1 -> 55.4).  What the lists hold is not known here: where routing leaves a tile of
// 128 rows no more than four chunks of 64 keys in all, the second group is a loss (1000 tokens, 32 / 8 heads, this launch alone, one
// group -> two: 1 chunk 9.6 -> 11.1 us, 2 10.8 -> 11.9, 3 11.9 -> 12.8, 4 13.2 -> 13.7; 5 14.5 -> 14.6, 6 15.7 -> 15.4, 9 19.3 -> 17.8, all
// 27.7 -> 23.3), most of it the larger workgroup's start: leaving such a list to the first group, without the exchange, gives
// 0.5 us back at 1 chunk, nothing at 2 and 3, and loses at 4.
static bool s2_paired(int64_t wgs, float tiles) { return wgs <= 256 && tiles > 4.f; }

// Parts a tile's chunk list is cut into at most.  512 workgroups are resident at once, two per CU
// (a single one on a CU runs 1.4 times as fast); fewer tiles than that leave the chip idle for as long
// as the longest list takes.  The number of parts is the one with the least estimated time, in units of
// a 64-key tile: rounds of resident workgroups times the tiles of a part, and for several parts 3 for the merge
// launch and 6 per round for the records.  Chunked prefill, whose lists are all about as long, is also cut
// where the tiles make two uneven rounds.  Measured, 8 kv-heads, group of 4, against a 32k cache, uncut -> cut:
// 65 tokens 707 -> 74 us, 300 709 -> 189, 700 718 -> 396, 1000 724 -> 500, 1500 850 -> 713, 2500 1449 -> 1190;
// whole prompts: 1 kv-head, 8000 tokens 195 -> 138, 2 kv-heads of one head, 12000 tokens 285 -> 152.
// Where the rule does not cut: 8 x 1000 tokens 33.2 -> 34.3 in two parts, 8 x 600 23.2 -> 26.7.  Two groups of waves (s2_paired)
// need no records and no second launch.  Their estimate, half the tiles and 8, says where they beat the cut, not what they gain over one
// group: near 256 workgroups (this launch alone, the best cut / two groups: 16 heads x 1024 tokens 25.9 / 24.2 us, x 1600
// 36.1 / 31.7, x 2048 47.1 / 39.6, 8 / 2 heads x 4096 66.0 / 63.5), while with fewer the cut is as fast or faster (16 tiles:
// 16 workgroups 22.3 / 23.4, 64 22.6 / 23.1 and 23.9 / 23.8; 21 tiles: 44 24.3 / 27.2, 88 26.3 / 27.5; 25 tiles: 104 27.8 / 31.1;
// 32 tiles: 64 26.6 / 37.5, 128 34.0 / 36.3; 40 tiles: 80 31.8 / 45.0, 160 37.9 / 43.4).
int s2_parts(const dash_params& p, const Layout& L) {
  if (!L.use_mfma) return 1;
  const int64_t wgs = (int64_t)s2_tiles(p, L) * p.h_kv * p.batch;
  if (wgs >= (L.pos0 >= p.n_q ? 1024 : 512)) return 1;
  const float tiles = (float)(L.t_all * (p.block_size >> 6));
  const int64_t most = s2_most_records(p, L);
  int best = 1;
  float best_cost = INFINITY;
  for (int n = 1; n * wgs <= (n == 1 ? wgs : most) && (n == 1 || n * kMinPartTiles <= tiles); n++) {
    const int64_t w = n * wgs, rest = w % 512;
    const float rounds = (float)(w / 512) + (rest == 0 ? 0.f : rest <= 256 ? 0.7f : 1.f);
    float cost = rounds * tiles / n + (n == 1 ? 0.f : 3.f + 6.f * w / 512);
    if (n == 1 && s2_paired(wgs, tiles)) cost = fminf(cost, 0.5f * tiles + 8.f);
    if (cost < best_cost) { best_cost = cost; best = n; }
  }
  return best;
}

static size_t s2_cnt_bytes(const dash_params& p, const Layout& L) {
  return ((size_t)s2_tiles(p, L) * p.h_kv * p.batch * 4 + 255) & ~(size_t)255;
}

// Records that s2_parts may ask for in a call of these parameters or in one with fewer queries, keys or
// sequences, so that a workspace made for the larger call serves the smaller one: parts of kMinPartTiles tiles
// each; and, from the costs above over all numbers of workgroups, no more than 256 below 24 tiles, 512 below 37 and 1024
// below 43 (a 1000-token prompt of 8 kv-heads, which is not cut itself: 17 MB at head dimension 128; one of up to
// 960 tokens: none).
static int64_t s2_most_records(const dash_params& p, const Layout& L) {
  const int tiles = L.t_all * (p.block_size >> 6);
  if (tiles < 2 * kMinPartTiles) return 0;
  const int64_t wgs = (int64_t)s2_tiles(p, L) * p.h_kv * p.batch, by_parts = wgs * (tiles / kMinPartTiles);
  const int by_cost = tiles < 24 ? 256 : tiles < 37 ? 512 : tiles < 43 ? 1024 : kMaxParts;
  return by_parts < by_cost ? by_parts : by_cost;
}
size_t s2_part_room(const dash_params& p, const Layout& L) {
  const int64_t n = s2_most_records(p, L);
  return n == 0 ? 0 : 1024 * 4 + (size_t)n * 128 * (p.head_dim + 2) * 4;     // counts of fewer than 1024 tiles
}

hipError_t launch_s2_mfma(const dash_params& p, const Layout& L, const void* q, const void* k,
                          const void* v, void* o, const uint32_t* mask, const float* bias,
                          char* part_ws, bool dense, hipStream_t st) {
  S2Args a;
  fill_s2_args(a, p, L, q, k, v, o, mask, bias);
  a.n_tiles = s2_tiles(p, L);
  if (L.s2_parts > 1) {
    a.max_parts = L.s2_parts;
    a.part_cnt = reinterpret_cast<int32_t*>(part_ws);
    a.part_ml = reinterpret_cast<float*>(part_ws + s2_cnt_bytes(p, L));
    a.part_o = a.part_ml + (size_t)a.n_tiles * a.hb * a.max_parts * 128 * 2;
  }
  const bool pair = a.max_parts == 1 && s2_paired((int64_t)a.n_tiles * a.hb, (float)(L.t_all * (p.block_size >> 6)));
  if (!dense && !pair && a.max_parts == 1 && s2_may_gather(a, p.head_dim)) s2_take_choice(a);
  if (p.head_dim == 128) return dense ? launch_s2_t<128, true>(a, pair, st) : launch_s2_t<128, false>(a, pair, st);
  return dense ? launch_s2_t<64, true>(a, pair, st) : launch_s2_t<64, false>(a, pair, st);
}

}  // namespace dash
