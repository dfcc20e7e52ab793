"""GPU parity at the sizes where the tilings change: the ranges of the decode step's kernels, the
128-key tiles and the cut row ranges of the backward pass, the 16-row tiles of the fp32 kernels.
Oracle and tolerances are those of parity_util and test_gpu_backward."""
import itertools

import numpy as np
import pytest
import torch

import parity_util as U
import test_gpu_backward as TB
from oracle import dash_oracle as orc
from paper_2605_18753_amd import binding as B
from paper_2605_18753_amd.inputs import Workload, make_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# One launch scores up to 640 chunks (320 for groups of 8 and 16) in the attention's workgroups when
# a pair has several splits; beyond that the scores have a launch of their own.
DECODE = [
    # name, batch, h_q, h_kv, n_kv, d, block, extra
    ("one_key", 2, 4, 2, 1, 128, 64, {}),
    ("own_chunk_only", 1, 8, 1, 64, 64, 64, {}),
    ("one_candidate", 1, 2, 2, 65, 128, 64, {}),
    ("16_candidates_and_one", 1, 8, 2, 17 * 64 + 1, 128, 64, {}),
    ("65_candidates_g1", 2, 2, 2, 65 * 64 + 33, 64, 64, {}),
    ("640_chunks_in_place", 1, 4, 1, 640 * 64 + 5, 64, 64, {"gamma": 1.5}),
    ("641_chunks_apart", 1, 4, 1, 641 * 64 + 5, 64, 64, {"gamma": 1.5}),
    ("g16_320_chunks_in_place", 1, 16, 1, 320 * 64 + 63, 128, 64, {"gamma": 2.0}),
    ("g8_321_chunks_apart", 1, 8, 1, 321 * 64 + 1, 128, 64, {"gamma": 2.0}),
    ("g16_apart_d64_b128_alpha3", 1, 16, 1, 400 * 128, 64, 128, {"alpha": 3.0}),
    ("2047_candidates_g2_alpha2", 1, 2, 1, 131072, 64, 64, {"alpha": 2.0, "gamma": 1.5}),
    # alpha > 2: up to 64 row slots per CU are solved in the attention's workgroups, more in a launch
    ("alpha3_512_chunks_one_per_cu", 1, 8, 1, 512 * 64 + 1, 64, 64, {"alpha": 3.0}),
    ("alpha3_513_chunks_in_a_launch", 1, 8, 1, 513 * 64 + 1, 64, 64, {"alpha": 3.0}),
    ("alpha25_g4_512_chunks_two_per_cu", 8, 4, 1, 512 * 64 + 63, 64, 64, {"alpha": 2.5, "window": 1}),
    ("alpha25_g8_257_chunks_in_a_launch", 8, 8, 1, 258 * 64, 64, 64, {"alpha": 2.5}),
    ("257_pairs_one_split", 257, 1, 1, 700, 64, 64, {}),
    ("171_pairs_alpha125", 57, 12, 3, 1500, 64, 64, {"alpha": 1.25, "window": 1}),
    ("alpha17_window8", 1, 4, 2, 3000, 128, 128, {"alpha": 1.7, "window": 8}),
]


@pytest.mark.parametrize("case", DECODE, ids=[c[0] for c in DECODE])
def test_decode_step(case):
    name, batch, h_q, h_kv, n_kv, d, block, extra = case
    w = Workload("edge_" + name, batch, h_q, h_kv, 1, n_kv, d, block, offset_sigma=0.7, seed=41, **extra)
    q, k, v = make_inputs(w, DEV)
    run = U.run_decode(w, q, k, v)
    heads = sorted({(b, r) for b in (0, batch // 2, batch - 1) for r in (0, h_kv - 1)})
    U.check_against_oracle(w, q, k, v, run, rows=[(b, r, 0) for b, r in heads])


@pytest.mark.parametrize("h_q,n_kv", [(16, 700 * 64 + 9), (4, 2000 * 64)])
def test_decode_without_room_for_score_rows(h_q, n_kv):
    """A workspace sized for a cache that keeps no score rows serves one that would: the step then
    routes in a launch of its own."""
    w = Workload("edge_small_ws", 1, h_q, 1, 1, n_kv, 64, 64, offset_sigma=0.7, gamma=1.5, seed=43)
    q, k, v = make_inputs(w, DEV)
    o = torch.full_like(q, float("nan"))
    p = B.make_params(q, k, v, o, w.block, w.alpha, w.gamma, w.sigma, True)
    kbar = torch.empty(B.kbar_shape(p), dtype=torch.float32, device=DEV)
    B.dash_kbar_compress(p, k, kbar)
    lists = B.Lists.allocate(p, DEV)
    ws = B.alloc_workspace(p, DEV)
    score_rows = h_q * ((n_kv // 64 + 15) // 16 * 16) * 4
    B.dash_attn_decode(p, q, k, v, kbar, o, lists, ws[:ws.numel() - (score_rows + 255) // 256 * 256])
    torch.cuda.synchronize()
    U.check_against_oracle(w, q, k, v, U.HipRun(o, kbar, lists, p))


def test_ragged_decode_replays_with_other_lengths():
    """A captured step keeps the number its split flags carry: every replay, with other lengths
    (other numbers of splits) each time, has to give what an uncaptured step gives."""
    w = Workload("edge_graph", 6, 8, 2, 1, 6000, 128, 64, offset_sigma=0.7, seed=44)
    q, k, v = make_inputs(w, DEV)
    o, want = torch.empty_like(q), torch.empty_like(q)
    p = B.make_params(q, k, v, o, w.block, w.alpha, w.gamma, w.sigma, True)
    kbar = torch.empty(B.kbar_shape(p), dtype=torch.float32, device=DEV)
    B.dash_kbar_compress(p, k, kbar)
    ws, ws2 = B.alloc_workspace(p, DEV), B.alloc_workspace(p, DEV)
    lens = torch.full((6,), 6000, dtype=torch.int32, device=DEV)
    step = lambda out, scratch: B.dash_attn_decode_ragged(p, q, k, v, kbar, lens, out, B.Lists(), scratch, update_cache=False)
    step(o, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(o, ws)
    for i in range(6):
        lens.copy_(torch.tensor([6000, 1 + 900 * i, 65 + i, 64 * (i + 1), 3000 - i, 5999], dtype=torch.int32))
        o.fill_(float("nan"))
        graph.replay()
        step(want, ws2)
        torch.cuda.synchronize()
        assert torch.equal(o, want), i


# 128-key tiles (the last one of 1, 64 and 65 keys), row ranges cut into parts, 16-row tiles of
# the fp32 kernels with ragged ends
BACKWARD = [
    ("b_129_b128", 1, 4, 2, 129, 128, 128, {"offset_sigma": 0.8}),
    ("b_257_mha", 2, 2, 2, 257, 64, 64, {"offset_sigma": 0.8}),
    ("b_193_b128", 1, 8, 1, 193, 128, 128, {"offset_sigma": 0.8}),
    ("b_parts_g16_d64", 1, 16, 1, 1037, 64, 64, {"offset_sigma": 0.8, "gamma": 2.0}),
    # among the 4608 rows of 1152 tokens one keeps a chunk 3e-6 above its threshold: 1/w = 1e11 there, and the chunk's
    # own bias gradient is 0 less the mean of all, so that its row shows what the mean is off by
    ("b_parts_noncausal_b128_near", 1, 4, 1, 1152, 128, 128, {"offset_sigma": 0.8, "causal": False}),
    ("b_parts_noncausal_b128", 1, 4, 1, 1280, 128, 128, {"offset_sigma": 0.8, "causal": False}),
    ("b_window3_alpha125_g2", 1, 2, 1, 831, 64, 64, {"offset_sigma": 0.8, "alpha": 1.25, "window": 3}),
    ("f_17", 1, 2, 1, 17, 64, 64, {"dtype": "fp32"}),
    ("f_g16_467_d128", 1, 16, 1, 467, 128, 64, {"dtype": "fp32", "offset_sigma": 0.8}),
    ("f_g8_331", 1, 8, 1, 331, 128, 64, {"dtype": "fp32", "offset_sigma": 0.8}),
]


@pytest.mark.parametrize("case", BACKWARD, ids=[c[0] for c in BACKWARD])
def test_backward(case):
    TB.test_backward_matches_the_oracle(case)


# rows of fewer than four chunks, and rows whose last four chunks do not begin at a multiple of four: the routing
# kernel reads them from up to three chunks before.  (Two and three chunks are not causal: a row with one candidate has no
# routing gradient, its bias gradient less the mean over that one being exactly 0, so that causal rows of two chunks have none
# and those of three 0.049 of the whole, by the oracle; the comparison asks for 0.05.)
@pytest.mark.parametrize("h_q,h_kv,chunks,d,extra", [
    (2, 1, 2, 64, {"causal": False}), (4, 1, 3, 128, {"causal": False}), (2, 2, 4, 64, {}), (1, 1, 5, 128, {"causal": False}), (4, 2, 6, 64, {"causal": False}),
    (1, 1, 7, 64, {"causal": False}), (2, 1, 17, 64, {"causal": False}), (1, 1, 18, 128, {}), (1, 1, 19, 64, {"causal": False}),
    (1, 1, 34, 64, {"gamma": 4.0})])              # lists across a mask word, waves that skip tiles
def test_backward_of_rows_of_any_number_of_chunks(h_q, h_kv, chunks, d, extra):
    TB.test_backward_matches_the_oracle((f"b_{chunks}_chunks", 1, h_q, h_kv, chunks * 64, d, 64, {"offset_sigma": 0.8, **extra}))


# one, two and three 64-key tiles, waves without rows, a group of 16 whose waves skip chunks
@pytest.mark.parametrize("h_q,h_kv,n,d,block,extra", [
    (4, 1, 65, 128, 64, {}), (16, 1, 129, 64, 64, {"gamma": 3.0}), (16, 1, 577, 128, 64, {"gamma": 4.0, "offset_sigma": 1.0}),
    (1, 1, 1025, 128, 128, {"gamma": 4.0, "offset_sigma": 1.0}), (2, 1, 999, 64, 64, {"window": 1, "sigma": 0.1})])
def test_prefill(h_q, h_kv, n, d, block, extra):
    w = Workload("edge_prefill", 1, h_q, h_kv, n, n, d, block, seed=45, **extra)
    q, k, v = make_inputs(w, DEV)
    U.check_against_oracle(w, q, k, v, U.run_prefill(w, q, k, v))


# Few tiles of queries against many chunks: the chunk list of a tile is cut into parts of at least 8
# tiles of 64 keys (the last part short, one part, a part per 8 tiles), merged by a kernel of its own.
@pytest.mark.parametrize("name,h_q,h_kv,n_q,n_kv,d,block,extra", [
    ("g4", 4, 1, 65, 64 * 150 + 65, 128, 64, {}),
    ("g1_window", 2, 2, 130, 64 * 70 + 130, 64, 64, {"window": 2}),
    ("g16_b128", 16, 1, 9, 128 * 40 + 64 + 9, 128, 128, {"gamma": 2.0}),
    ("g8_sparse", 8, 1, 33, 64 * 301 + 33, 64, 64, {"gamma": 4.0, "offset_sigma": 1.0}),
    ("g2_seventeen_chunks", 4, 2, 63, 64 * 16 + 63, 128, 64, {"alpha": 2.0}),
    # rows of 255 .. 257, 511 .. 513 and 255 .. 513 candidates: the routing kernels' ranges, in one launch
    ("rows_of_256", 4, 1, 130, 64 * 255 + 130, 64, 64, {"gamma": 2.0}),
    ("rows_of_512", 8, 1, 130, 64 * 511 + 130, 128, 64, {"gamma": 2.0}),
    ("rows_of_512_d64", 2, 1, 130, 64 * 511 + 130, 64, 64, {"gamma": 1.5}),
    ("noncausal", 4, 2, 1024, 1024, 128, 64, {"causal": False})])
def test_prefill_cut_chunk_lists(name, h_q, h_kv, n_q, n_kv, d, block, extra):
    w = Workload("edge_cut_" + name, 1, h_q, h_kv, n_q, n_kv, d, block, seed=46, **extra)
    q, k, v = make_inputs(w, DEV)
    run = U.run_prefill(w, q, k, v)
    rows = None if n_q * n_kv < 1 << 20 else U.sample_rows(w, 60)
    U.check_against_oracle(w, q, k, v, run, rows=rows)
    o = torch.full_like(q, float("nan"))
    ws = B.alloc_workspace(run.params, DEV)
    # the dense reference is cut the same way
    B.dense_attn(run.params, q, k, v, o, ws)
    torch.cuda.synchronize()
    qf, kf, vf = (t.double().cpu() for t in (q, k, v))
    g, pos = h_q // h_kv, torch.arange(n_kv - n_q, n_kv)
    for h in range(h_q):
        z = qf[0, h] @ kf[0, h // g].T / d ** 0.5
        if w.causal:
            z.masked_fill_(torch.arange(n_kv)[None, :] > pos[:, None], float("-inf"))
        ref = torch.softmax(z, -1) @ vf[0, h // g]
        assert (o[0, h].double().cpu() - ref).abs().max() <= 2e-2 * ref.abs().max()


# Two groups of waves walk the halves of a tile's chunk list where at most 256 tiles are not cut and have more than four tiles of 64
# keys: an even and an odd number of chunks, chunks of two tiles, tiles with fewer chunks than groups, waves without rows, the last launch
# of 256 tiles and the first of more, sparse rows whose second half is the own chunk alone.
@pytest.mark.parametrize("name,batch,h_q,h_kv,n,d,block,extra", [
    ("four_tiles", 1, 4, 2, 256, 128, 64, {}), ("five_tiles", 1, 4, 2, 257, 128, 64, {}), ("six_tiles_b128", 2, 2, 1, 321, 64, 128, {}),
    ("ragged_g16", 1, 16, 1, 577, 64, 64, {"gamma": 2.0}), ("window", 1, 8, 8, 390, 128, 64, {"window": 2}),
    ("256_tiles", 32, 1, 1, 1024, 64, 64, {"gamma": 2.0}),
    ("264_tiles", 33, 1, 1, 1024, 64, 64, {"gamma": 2.0}), ("sparse_g1", 1, 2, 2, 950, 128, 64, {"gamma": 4.0, "offset_sigma": 1.0}),
    ("noncausal", 1, 8, 8, 832, 128, 64, {"causal": False}),
    # every chunk kept: behind the last bias of the last token the array ends
    ("noncausal_all", 1, 2, 1, 640, 128, 64, {"causal": False, "gamma": 0.01})])
def test_prefill_in_two_groups(name, batch, h_q, h_kv, n, d, block, extra):
    w = Workload("edge_pair_" + name, batch, h_q, h_kv, n, n, d, block, seed=49, **{"offset_sigma": 0.7, **extra})
    q, k, v = make_inputs(w, DEV)
    run = U.run_prefill(w, q, k, v)
    U.check_against_oracle(w, q, k, v, run, rows=U.sample_rows(w, 80) if batch > 2 else None)
    check_dense_uncut(w, run.params, q, k, v)


def check_dense_uncut(w, p, q, k, v):
    """dense_attn against fp64, in a launch that is not cut into parts: the records of parts are all that it
    writes into the workspace."""
    o, ws = torch.full_like(q, float("nan")), B.alloc_workspace(p, DEV).fill_(0xA5)
    B.dense_attn(p, q, k, v, o, ws)
    torch.cuda.synchronize()
    assert bool((ws == 0xA5).all()), "cut into parts: not the kernels this is about"
    g, pos = w.h_q // w.h_kv, torch.arange(w.n_q)
    for b in {0, w.batch - 1}:
        for h in range(w.h_q):
            z = q[b, h].double().cpu() @ k[b, h // g].double().cpu().T / w.head_dim ** 0.5
            if w.causal:
                z.masked_fill_(pos[None, :] > pos[:, None], float("-inf"))
            ref = torch.softmax(z, -1) @ v[b, h // g].double().cpu()
            assert (o[b, h].double().cpu() - ref).abs().max() <= 2e-2 * ref.abs().max()   # the bar of the cut lists' test


@pytest.mark.parametrize("h_q,n_q,chunks,d,block", [(4, 64, 33, 128, 64), (4, 64, 2048, 64, 64), (2, 130, 2048, 64, 128), (16, 40, 64, 64, 64)])
def test_attention_over_lists_at_word_edges(h_q, n_q, chunks, d, block):
    """Lists whose chunks lie at the edges of mask bytes and words, up to the longest sequence (4096
    tiles of 64 keys), other ones for every token; reference in fp32."""
    n_kv = n_q + (chunks * block - n_q) // 64 * 64
    w = Workload("edge_lists", 1, h_q, 1, n_q, n_kv, d, block, seed=53)
    q, k, v = make_inputs(w, DEV)
    o = torch.empty_like(q)
    p = B.make_params(q, k, v, o, block)
    t_all, pos = B.list_stride(p), n_kv - n_q + torch.arange(n_q, device=DEV)
    edge = [c for c in (0, 1, 7, 8, 31, 32, 33, 62, 63, 64, 1023, 1024, 2015, 2016, 2046) if c < t_all]
    keep = torch.zeros((n_q, t_all), dtype=torch.bool, device=DEV)
    for i, c in enumerate(edge):
        keep[:, c] = (torch.arange(n_q, device=DEV) // 3 + i) % 3 != 0
    own = pos // block
    keep &= torch.arange(t_all, device=DEV)[None] < own[:, None]
    keep[torch.arange(n_q), own] = True
    words = B.mask_words(p)
    bits = torch.nn.functional.pad(keep, (0, words * 32 - t_all)).view(n_q, words, 32).to(torch.int64)
    mask = (bits << torch.arange(32, device=DEV)).sum(-1)
    mask = torch.where(mask >= 1 << 31, mask - (1 << 32), mask).to(torch.int32).view(1, 1, n_q, words)
    by_chunk = torch.randn((n_q, t_all), device=DEV)
    by_chunk[torch.arange(n_q), own] = 0.0
    bias = torch.zeros((1, 1, n_q, t_all), device=DEV)
    for t in range(n_q):
        row = by_chunk[t, keep[t]]
        bias[0, 0, t, :row.numel()] = row
    B.dash_stage2_attend(p, q, k, v, o, B.Lists(mask=mask.contiguous(), bias=bias), B.alloc_workspace(p, DEV))
    add = torch.where(keep, by_chunk, torch.full_like(by_chunk, float("-inf"))).repeat_interleave(block, 1)[:, :n_kv]
    add = torch.where(torch.arange(n_kv, device=DEV)[None] <= pos[:, None], add, torch.full_like(add, float("-inf")))
    ref = torch.softmax(q[0].float() @ k[0, 0].float().T / d ** 0.5 + add[None], -1) @ v[0, 0].float()
    err = ((o[0].float() - ref).abs().amax(-1) / ref.abs().amax()).max().item()
    print(f"[parity] lists at word edges {chunks} x {block}: {err:.2e}")
    assert err <= 2e-2, err


def random_lists(p, n_q, n_kv, block, causal, sparsity, seed):
    """Lists of chunks kept at random, with a token of every chunk and a chunk of every token of a stretch; without a causal mask
    a token of no chunk."""
    t_all, words = B.list_stride(p), B.mask_words(p)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    c = torch.arange(words * 32, device=DEV)
    keep = torch.rand((p.batch, p.h_kv, n_q, words * 32), generator=gen, device=DEV) >= sparsity
    keep[:, :, n_q // 2 + 5] = True
    keep[:, :, n_q // 3: n_q // 3 + 300, 7] = True
    keep[:, :, n_q // 4 + 3] &= causal
    own = ((n_kv - n_q + torch.arange(n_q, device=DEV)) // block).view(1, n_q, 1)
    keep = (keep & (c < own)) | (c == own) if causal else keep & (c < t_all)
    mask = torch.zeros((p.batch, p.h_kv, n_q, words), dtype=torch.int64, device=DEV)
    for i in range(32):
        mask |= keep.view(p.batch, p.h_kv, n_q, words, 32)[..., i].to(torch.int64) << i
    mask = torch.where(mask >= 1 << 31, mask - (1 << 32), mask).to(torch.int32)
    return B.Lists(mask=mask, bias=torch.randn((p.batch, p.h_kv, n_q, t_all), generator=gen, device=DEV)), keep


def gathers_rows(p, q, k, v, o, keep, r, lists, expected):
    """Which of the two kernels takes the launch whose output is o.  In the one that walks the union of a wave's tokens an infinity in a value
    reaches all rows of the wave (0 times infinity is a NaN); the one that gathers rows has it reach the tokens that kept the chunk.
    keep: tokens x chunks of kv-head r of the first sequence."""
    chunk = int(keep[:, :keep.shape[1] // 2].sum(0).argmax()) if expected else keep.shape[1] // 8
    other = ~keep[:, chunk]
    assert bool(other.any()) and bool(keep[:, chunk].any())
    g = q.shape[1] // v.shape[1]
    got = torch.empty_like(o)
    for t in ("k", "v"):
        kk, vv = k.clone(), v.clone()
        (kk if t == "k" else vv)[0, r, chunk * p.block_size + 5] = float("nan" if t == "k" else "inf")
        B.dash_stage2_attend(p, q, kk, vv, got, lists, B.alloc_workspace(p, DEV))
        far, was = got[0, r * g:(r + 1) * g][:, other], o[0, r * g:(r + 1) * g][:, other]
        assert bool(torch.isfinite(was.float()).all())
        same = torch.equal(far, was)
        assert same == expected, (t, chunk)


GATHERED = [
    # name, h_q, h_kv, n_q, n_kv, d, block, causal, sparsity, interleaved, batch (1): at least 320000 tiles of 128 rows x 64 keys
    ("g4_odd_tail", 32, 8, 2000, 44240, 128, 64, True, 0.97, False),
    ("g4_interleaved_b128", 32, 8, 4097, 4097 + 64 * 300, 128, 128, True, 0.95, True),
    ("g4_d64_dense", 32, 8, 2000, 44240, 64, 64, True, 0.3, False),
    ("g1_d64", 32, 32, 13001, 13001, 64, 64, True, 0.93, False),
    ("g1_noncausal", 16, 16, 13056, 13056, 128, 128, False, 0.9, False),
    ("g2_d64_interleaved", 16, 8, 18432, 18432, 64, 64, True, 0.95, True),
    ("g2_one_token_over", 32, 16, 12865, 12865, 128, 64, True, 0.9, False),
    ("g8", 32, 4, 12901, 12901, 128, 64, True, 0.985, False),
    ("g4_d64", 32, 8, 2000, 44240, 64, 64, True, 0.97, False),
    ("g8_d64_interleaved", 32, 4, 12901, 12901, 64, 64, True, 0.985, True),
    ("g4_two_sequences", 16, 4, 2000, 44240, 128, 64, True, 0.97, False, 2),
]


@pytest.mark.parametrize("case", GATHERED, ids=[c[0] for c in GATHERED])
def test_attention_over_gathered_rows(case):
    """Launches large enough to be left to the kernel that gathers the rows of a chunk; tokens that keep every chunk, and chunks that
    every token of a stretch keeps, among sparse ones; logits that grow along the keys.  Reference in fp64 on sampled tokens.  The bar is
    that of the other given lists."""
    name, h_q, h_kv, n_q, n_kv, d, block, causal, sparsity, interleaved, batch = (*case, 1)[:11]
    w = Workload("gathered_" + name, batch, h_q, h_kv, n_q, n_kv, d, block, causal=causal, seed=57)
    q, k, v = make_inputs(w, DEV)
    k *= torch.linspace(0.5, 3.0, n_kv, device=DEV).view(1, 1, n_kv, 1).to(k.dtype)
    if interleaved:                              # [batch, token, head, d] in memory
        q, k, v = (x.transpose(1, 2).contiguous().transpose(1, 2) for x in (q, k, v))
    o = torch.full_like(q, float("nan"))
    p = B.make_params(q, k, v, o, block, causal=causal)
    lists, keep = random_lists(p, n_q, n_kv, block, causal, sparsity, 58)
    t_all = B.list_stride(p)
    ws = B.alloc_workspace(p, DEV).fill_(0xA5)
    B.dash_stage2_attend(p, q, k, v, o, lists, ws)
    # an uncut launch over lists of the caller's uses nothing of the workspace, which other calls may be using
    assert bool((ws == 0xA5).all())
    gathers_rows(p, q, k, v, o, keep[0, h_kv - 1], h_kv - 1, lists, sparsity >= 0.5)
    again = torch.empty_like(o)
    B.dash_stage2_attend(p, q, k, v, again, lists, ws)
    assert torch.equal(o, again)
    # a NaN in a query reaches that row.  The rows that a wave holds together raise their reference maxima together, so P of its neighbours may be
    # rounded at another scale: each of the two results is within the bar of the exact one
    bad = q.clone()
    bad[0, h_q - 1, n_q // 2 + 5] = float("nan")
    B.dash_stage2_attend(p, bad, k, v, again, lists, ws)
    hit = torch.isnan(again.float())
    assert bool(hit[0, h_q - 1, n_q // 2 + 5].all()) and int(hit.sum()) == d
    assert bool(((o - again)[~hit].abs() <= 2 * 2e-2 * o.abs().max()).all())
    g, worst = h_q // h_kv, 0.0
    toks = sorted({0, 1, 63, 64, n_q // 3 + 17, n_q // 2 + 4, n_q // 2 + 5, n_q // 2 + 6, n_q - 2, n_q - 1} | {(i * 977) % n_q for i in range(20)})
    assert bool(torch.isfinite(o.float()).all())
    if not causal:
        assert bool((o[:, :, n_q // 4 + 3] == 0).all())
    for s, r in itertools.product(range(batch), range(h_kv)):
        for t in toks:
            pos = n_kv - n_q + t
            kept = keep[s, r, t, :t_all]
            add = torch.full((t_all,), float("-inf"), device=DEV, dtype=torch.float64)
            add[kept] = lists.bias[s, r, t, :int(kept.sum())].double()
            if causal:
                add[pos // block] = 0.0
            add = add.repeat_interleave(block)[:n_kv]
            if causal:
                add[pos + 1:] = float("-inf")
            j = add > float("-inf")
            z = q[s, r * g:(r + 1) * g, t].double() @ k[s, r, j].double().T / d ** 0.5 + add[j]
            ref = torch.softmax(z, -1) @ v[s, r, j].double()
            worst = max(worst, ((o[s, r * g:(r + 1) * g, t].double() - ref).abs().max() / ref.abs().max()).item())
    print(f"[parity] gathered rows {name}: {worst:.2e}")
    assert worst <= 2e-2, worst


@pytest.mark.parametrize("batch,h_q,h_kv,n_q,n_kv,d", [(1, 32, 8, 2000, 44240, 128), (2, 16, 2, 2003, 44243, 64)])
def test_gathered_rows_behind_the_end_of_a_padded_buffer(batch, h_q, h_kv, n_q, n_kv, d):
    """NaN behind the last token of every head of a larger buffer, with a last chunk that is not full: nobody reads it."""
    q, k, v = make_inputs(Workload("gathered_padded", batch, h_q, h_kv, n_q, n_kv, d, 64, seed=61), DEV)
    p = B.make_params(q, k, v, torch.empty_like(q), 64)
    lists, keep = random_lists(p, n_q, n_kv, 64, True, 0.985, 62)

    def padded(x):
        big = torch.full((*x.shape[:2], x.shape[2] + 40, d), float("nan"), dtype=x.dtype, device=DEV)
        big[:, :, :x.shape[2]] = x
        return big[:, :, :x.shape[2]]

    out = []
    for qq, kk, vv in ((q, k, v), (padded(q), padded(k), padded(v))):
        o = torch.full_like(q, float("nan"))
        pp = B.make_params(qq, kk, vv, o, 64)
        B.dash_stage2_attend(pp, qq, kk, vv, o, lists, B.alloc_workspace(pp, DEV))
        out.append(o)
    gathers_rows(p, q, k, v, out[0], keep[0, h_kv - 1], h_kv - 1, lists, True)
    assert bool(torch.isfinite(out[1].float()).all())
    assert torch.equal(out[0], out[1])


def test_prefill_that_gathers_rows():
    """The whole prefill, two sequences, a window beside the routed chunks.  Oracle and tolerances are those of the other prefills."""
    w = Workload("gathered_prefill", 2, 16, 4, 12901, 12901, 128, 64, alpha=2.0, gamma=4.0, window=1, offset_sigma=1.0, seed=63)
    q, k, v = make_inputs(w, DEV)
    run = U.run_prefill(w, q, k, v)
    rep, _ = U.check_against_oracle(w, q, k, v, run, rows=U.sample_rows(w, 24, heads=[(0, 0), (0, 3), (1, 1)]))
    print(f"[parity] gathered prefill: sparsity {rep.sparsity:.3f} {rep.errors()}")
    keep = torch.stack([(run.lists.mask[0, 3, :, c // 32] >> (c % 32)) & 1 for c in range(B.list_stride(run.params))], 1).bool()
    gathers_rows(run.params, q, k, v, run.o, keep, 3, run.lists, True)


def sparse_and_dense(h_q=32, h_kv=4, n=12901, d=64):
    """Inputs of a launch that either kernel may take, lists that leave it to one or the other, and what they give."""
    q, k, v = make_inputs(Workload("gathered_choice", 1, h_q, h_kv, n, n, d, 64, seed=59), DEV)
    p = B.make_params(q, k, v, torch.empty_like(q), 64)
    ws = B.alloc_workspace(p, DEV)
    lists, want = [], []
    for sparsity in (0.985, 0.4):
        ls, keep = random_lists(p, n, n, 64, True, sparsity, 60)
        o = torch.empty_like(q)
        B.dash_stage2_attend(p, q, k, v, o, ls, ws)
        gathers_rows(p, q, k, v, o, keep[0, 0], 0, ls, sparsity > 0.9)
        lists.append(ls)
        want.append(o)
    return p, q, k, v, ws, lists, want


@pytest.mark.parametrize("first", [0, 1])
@pytest.mark.parametrize("calls", [8, 64])
def test_uncut_launches_share_a_workspace(calls, first):
    """Launches over lists of the caller's on two streams, of either kernel: they keep nothing in the workspace.  64 on each
    stream use every record of a choice twice, and two in flight may meet in one."""
    p, q, k, v, ws, lists, want = sparse_and_dense()
    got = [[torch.full_like(q, float("nan")) for _ in range(calls)] for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for st in streams:
        with torch.cuda.stream(st):
            torch.cuda._sleep(20_000_000)        # the calls are there before the first begins
    for which in (first, 1 - first):
        with torch.cuda.stream(streams[which]):
            for i in range(calls):
                B.dash_stage2_attend(p, q, k, v, got[which][i], lists[which], ws)
    torch.cuda.synchronize()
    bits = [sum(torch.equal(o, want[which]) for o in got[which]) for which in range(2)]
    print(f"[choice] {calls} calls on each of two streams, of the same bits as alone: {bits}")
    assert bits[0] == calls and (calls > 32 or bits[1] == calls)
    # a launch that does not know its choice is attended by both kernels; the bar is that of the other given lists
    bar = 2e-2 * want[1].abs().max()
    for o in got[1]:
        assert bool(((o - want[1]).abs() <= bar).all())


def test_a_captured_launch_chooses_its_kernel_at_every_replay():
    p, q, k, v, ws, lists, want = sparse_and_dense()
    mask, bias, o = lists[0].mask.clone(), lists[0].bias.clone(), torch.empty_like(q)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.dash_stage2_attend(p, q, k, v, o, B.Lists(mask=mask, bias=bias), ws)
    for i in (0, 1, 1, 0, 1, 0):
        mask.copy_(lists[i].mask)
        bias.copy_(lists[i].bias)
        o.fill_(float("nan"))
        graph.replay()
        again = torch.empty_like(q)
        B.dash_stage2_attend(p, q, k, v, again, lists[1 - i], ws)
        torch.cuda.synchronize()
        assert torch.equal(o, want[i]) and torch.equal(again, want[1 - i]), i


@pytest.mark.parametrize("h,n,d,block", [(8, 832, 128, 64), (2, 512, 64, 64), (4, 896, 64, 128)])
def test_attention_of_tiles_that_keep_one_chunk(h, n, d, block):
    """Two groups of waves over lists of a single chunk: the second group's half is empty.  Reference in fp32."""
    w = Workload("edge_one_chunk", 1, h, h, n, n, d, block, causal=False, seed=55)
    q, k, v = make_inputs(w, DEV)
    o = torch.full_like(q, float("nan"))
    p = B.make_params(q, k, v, o, block, causal=False)
    chunk = (torch.arange(n, device=DEV) // 128 * 5 + 3) % (n // block)          # one of every 128 rows
    words = B.mask_words(p)
    mask = torch.zeros((1, h, n, words), dtype=torch.int64, device=DEV)
    mask[:, :, torch.arange(n, device=DEV), chunk // 32] = 1 << (chunk % 32)
    bias = torch.randn((1, h, n, B.list_stride(p)), device=DEV)
    B.dash_stage2_attend(p, q, k, v, o, B.Lists(mask=mask.to(torch.int32), bias=bias), B.alloc_workspace(p, DEV))
    key = chunk[:, None] * block + torch.arange(block, device=DEV)
    z = (q[0].float()[:, :, None] * k[0].float()[:, key]).sum(-1) / d ** 0.5
    ref = (torch.softmax(z, -1)[..., None] * v[0].float()[:, key]).sum(2)
    err = ((o[0].float() - ref).abs().amax(-1) / ref.abs().amax()).max().item()
    print(f"[parity] tiles of one chunk {h} x {n}: {err:.2e}")
    assert err <= 2e-2, err


# logits that rise or fall by a factor of four along the keys: a late raise of the running maximum, and two groups of waves
# whose maxima lie far apart, either way round; launches of three workgroups per CU
@pytest.mark.parametrize("first,last", [(1.0, 4.0), (4.0, 1.0)])
@pytest.mark.parametrize("name,batch,h_q,h_kv,n,d", [("two_groups", 1, 8, 8, 832, 128), ("two_groups_d64", 1, 16, 2, 832, 64), ("one_group", 33, 1, 1, 1000, 128),
                                                        ("three_per_cu", 103, 1, 1, 1000, 64), ("three_per_cu_g4", 26, 4, 1, 1001, 64)])
def test_prefill_of_rising_and_falling_logits(name, batch, h_q, h_kv, n, d, first, last):
    w = Workload("edge_ramp_" + name, batch, h_q, h_kv, n, n, d, 64, seed=50, offset_sigma=0.3)
    q, k, v = make_inputs(w, DEV)
    k = (k.float() * torch.linspace(first, last, n, device=DEV).view(1, 1, n, 1)).to(k.dtype)
    q = (q.float() * 3.0).to(q.dtype)
    run = U.run_prefill(w, q, k, v)
    U.check_against_oracle(w, q, k, v, run, rows=U.sample_rows(w, 96))
    check_dense_uncut(w, run.params, q, k, v)


@pytest.mark.parametrize("batch,h_q,h_kv,n_kv,extra", [
    (1, 8, 2, 1000, {}), (2, 16, 1, 400 * 64 + 7, {"gamma": 2.0}), (1, 4, 1, 700 * 64, {"gamma": 1.5, "window": 2}), (300, 2, 2, 300, {})])
def test_decode_keeps_its_lists_in_the_workspace(batch, h_q, h_kv, n_kv, extra):
    """Lists that are not asked for stay in the workspace for dash_stage2_attend, as those of
    dash_stage1_route do.  The workspace first holds the lists of other queries."""
    w = Workload("edge_ws_lists", batch, h_q, h_kv, 1, n_kv, 64, 64, offset_sigma=1.0, seed=47, **extra)
    q, k, v = make_inputs(w, DEV)
    o, again = torch.empty_like(q), torch.empty_like(q)
    p = B.make_params(q, k, v, o, w.block, w.alpha, w.gamma, 1e6, True, window=w.window)
    kbar = torch.empty(B.kbar_shape(p), dtype=torch.float32, device=DEV)
    B.dash_kbar_compress(p, k, kbar)
    ws = B.alloc_workspace(p, DEV)
    B.dash_stage1_route(p, -q, kbar, B.Lists(), ws)
    B.dash_attn_decode(p, q, k, v, kbar, o, B.Lists(), ws)
    B.dash_stage2_attend(p, q, k, v, again, B.Lists(), ws)
    torch.cuda.synchronize()
    # the same kernel on the same splits
    assert torch.equal(o, again)


# Per-sequence lengths: the splits of a kv-head are dealt to the sequences 64 at a time, by length or,
# over lists in memory, by what the lists hold.
@pytest.mark.parametrize("name,batch,h_q,h_kv,n_kv,d,block,cut,extra", [
    ("more_than_two_rounds", 130, 2, 1, 1500, 64, 64, 0, {}),
    ("one_split_left_over", 65, 4, 4, 900, 128, 64, 0, {"window": 1}),
    ("some_have_two", 40, 16, 8, 700, 64, 64, 0, {}),
    ("no_slot_to_spare", 520, 1, 1, 300, 64, 64, 0, {}),
    ("lists", 70, 8, 1, 400 * 64 + 9, 64, 64, "scores", {"gamma": 2.0}),
    ("lists_few_sequences", 3, 16, 1, 350 * 128 + 77, 128, 128, "scores", {"gamma": 2.0, "window": 2}),
    ("lists_200_pairs", 100, 16, 2, 321 * 64 + 1, 64, 64, "scores", {"gamma": 3.0}),
    # more summaries than score rows are kept for
    ("lists_one_split_each", 257, 16, 1, 1060 * 64, 64, 64, 0, {"gamma": 4.0})])
def test_ragged_decode_deals_its_splits(name, batch, h_q, h_kv, n_kv, d, block, cut, extra):
    w = Workload("edge_ragged_" + name, batch, h_q, h_kv, 1, n_kv, d, block, offset_sigma=0.7, seed=48, **extra)
    q, k, v = make_inputs(w, DEV)
    o = torch.full_like(q, float("nan"))
    p = B.make_params(q, k, v, o, block, w.alpha, w.gamma, w.sigma, True, window=w.window)
    kbar = torch.empty(B.kbar_shape(p), dtype=torch.float32, device=DEV)
    B.dash_kbar_compress(p, k, kbar)
    rng = np.random.default_rng(49)
    lens = np.where(rng.random(batch) < 0.5, rng.integers(1, n_kv + 1, batch), rng.integers(1, min(n_kv, 200) + 1, batch))
    lens[[0, -1]] = 1, n_kv
    lists, ws = B.Lists.allocate(p, DEV), B.alloc_workspace(p, DEV)
    if cut == "scores":                           # a workspace without its score rows: routing in a launch of its own
        cut = (batch * h_q * ((n_kv // block + 15) // 16 * 16) * 4 + 255) // 256 * 256
    ws = ws[:ws.numel() - cut]
    B.dash_attn_decode_ragged(p, q, k, v, kbar, torch.tensor(lens, dtype=torch.int32, device=DEV), o, lists, ws, update_cache=False)
    torch.cuda.synchronize()
    prm, g, rep = U.oracle_params(w), h_q // h_kv, U.SupportReport()
    longest = int(np.argsort(lens)[-2])
    for b in sorted({i for i in (0, 1, 62, 63, 64, 65, 127, 128, 129, batch // 2, longest, batch - 2, batch - 1) if i < batch}):
        n = int(lens[b])
        for r in {0, h_kv - 1}:
            kn, vn = U.to_np(k[b, r, :n]), U.to_np(v[b, r, :n])
            rr = orc.dash_row_at(U.to_np(q[b, r * g:(r + 1) * g, 0]), kn, vn, orc.block_mean_summaries(kn, block), prm, n - 1, (b, r, 0))
            U.compare_row(rr, w, lists.mask[b, r, 0].cpu().numpy(), int(lists.cnt[b, r, 0]), lists.idx[b, r, 0].cpu().numpy(),
                          lists.bias[b, r, 0].cpu().numpy(), lists.tau[b, r * g:(r + 1) * g, 0].cpu().numpy(), rep, B.list_stride(p))
            got = U.to_np(o[b, r * g:(r + 1) * g, 0]).astype(np.float64)
            assert np.abs(got - rr.o).max() <= 2e-2 * np.abs(rr.o).max(), (b, r)
    assert rep.mismatched == 0 and rep.exempt <= 1
    # every sequence was written
    assert not bool(torch.isnan(o.float()).any())


def test_routing_needs_no_room_for_records():
    """dash_stage1_route writes none of the records of cut chunk lists."""
    w = Workload("edge_route_ws", 1, 8, 2, 1024, 1024, 128, 64, offset_sigma=0.7, seed=50)
    q, k, v = make_inputs(w, DEV)
    run = U.run_prefill(w, q, k, v)
    lists, ws = B.Lists.allocate(run.params, DEV), B.alloc_workspace(run.params, DEV)
    pieces, mask, bias = 2 * 16 * 3 * 128 * 2, 2 * 1024 * 4, 2 * 1024 * 16 * 4       # all multiples of 256
    assert pieces + mask + bias + 256 < ws.numel()
    B.dash_stage1_route(run.params, q, run.kbar, lists, ws[:pieces + mask + bias + 256])
    torch.cuda.synchronize()
    for name in ("mask", "cnt", "idx", "tau"):
        assert torch.equal(getattr(lists, name), getattr(run.lists, name)), name


# Tensors in other layouts: tokens before heads, and heads of a larger padded buffer.  The kernels read and write
# the same values in the same order, so the results are those of contiguous tensors, bit for bit.
@pytest.mark.parametrize("layout", ["token_major", "padded"])
@pytest.mark.parametrize("name,h_q,h_kv,n_q,n_kv,d,block,extra", [
    ("cut_lists_g4", 8, 2, 65, 64 * 150 + 65, 128, 64, {}), ("cut_lists_g1_d64", 2, 2, 130, 64 * 70 + 130, 64, 64, {"window": 2}),
    ("cut_lists_g16_b128", 16, 1, 9, 128 * 40 + 64 + 9, 128, 128, {"gamma": 2.0}),
    ("decode_in_place", 8, 2, 1, 1000, 128, 64, {}), ("decode_scores_apart", 4, 1, 1, 641 * 64 + 5, 64, 64, {"gamma": 1.5}),
    ("decode_scores_apart_g16", 16, 1, 1, 400 * 128 + 3, 128, 128, {"gamma": 2.0}), ("decode_one_split", 4, 1, 1, 300, 64, 64, {})])
def test_other_layouts(layout, name, h_q, h_kv, n_q, n_kv, d, block, extra):
    batch = 260 if name == "decode_one_split" else 2
    w = Workload("edge_layout_" + name, batch, h_q, h_kv, n_q, n_kv, d, block, offset_sigma=0.7, seed=55, **extra)
    q, k, v = make_inputs(w, DEV)

    def relaid(t):
        b, h, n, _ = t.shape
        if layout == "token_major":
            out = torch.empty(b, n, h, d, dtype=t.dtype, device=DEV).transpose(1, 2)
        else:
            out = torch.full((b + 1, h + 1, n + 24, d), float("nan"), dtype=t.dtype, device=DEV)[1:, 1:, 16:16 + n]
        return out.copy_(t)

    def results(q, k, v):
        o, dense = relaid(torch.zeros_like(q)), relaid(torch.zeros_like(q))
        if q.is_contiguous():
            o, dense = torch.empty_like(q), torch.empty_like(q)
        p = B.make_params(q, k, v, o, block, w.alpha, w.gamma, w.sigma, True, window=w.window)
        kbar = torch.empty(B.kbar_shape(p), dtype=torch.float32, device=DEV)
        lists, ws = B.Lists.allocate(p, DEV), B.alloc_workspace(p, DEV)
        if n_q == 1:
            B.dash_kbar_compress(p, k, kbar)
            B.dash_attn_decode(p, q, k, v, kbar, o, lists, ws)
        else:
            B.dash_attn_prefill(p, q, k, v, o, kbar, lists, ws)
        B.dense_attn(p, q, k, v, dense, ws)
        torch.cuda.synchronize()
        return dict(o=o, dense=dense, kbar=kbar, mask=lists.mask, cnt=lists.cnt, tau=lists.tau)

    want, got = results(q, k, v), results(relaid(q), relaid(k), relaid(v))
    for key in want:
        assert torch.equal(got[key], want[key]), key
    assert bool(torch.isfinite(want["o"].float()).all())


@pytest.mark.parametrize("h_q,h_kv,n_q,chunks,d,extra", [
    (4, 1, 300, 384, 128, {}),                      # the last rows whose scores fill 24 register slots, then 32
    (16, 1, 200, 384, 64, {"gamma": 2.0}),
    (1, 1, 400, 384, 128, {"alpha": 3.0}),
    (4, 2, 300, 768, 128, {"window": 1}),           # the same on wave pairs
    (8, 1, 200, 768, 128, {"alpha": 1.25}),
])
def test_routing_row_length_steps(h_q, h_kv, n_q, chunks, d, extra):
    """Rows with `chunks` candidates and with one more, whose kernels hold another number of scores per lane."""
    first = (chunks + extra.get("window", 0) + 1) * 64 - 128
    w = Workload(f"edge_row_{chunks}_{h_q}_{d}", 1, h_q, h_kv, n_q, first + n_q, d, 64, offset_sigma=0.7, seed=67, **extra)
    q, k, v = make_inputs(w, DEV)
    run = U.run_prefill(w, q, k, v)
    toks = [0, 127, 128, n_q - 1]                   # token 128 is the first with one candidate more
    U.check_against_oracle(w, q, k, v, run, rows=[(0, r, i) for r in range(h_kv) for i in toks])


@pytest.mark.parametrize("h_q,h_kv,chunks,alpha", [(1, 1, 1024, 1.5), (2, 2, 1500, 1.5), (1, 1, 1100, 1.25), (1, 1, 1100, 2.0),
                                                   (2, 1, 1024, 1.5), (4, 1, 1400, 1.5), (16, 1, 1024, 1.5)])
def test_routing_of_rows_of_more_than_1024_chunks(h_q, h_kv, chunks, alpha):
    """Every group size and exponent; rows in every quarter of a wave's lanes, in both of a workgroup's chunks."""
    w = Workload(f"edge_long_{chunks}_{h_q}_{alpha}", 1, h_q, h_kv, 200, (chunks - 1) * 64 + 200, 128, 64, offset_sigma=0.7, seed=68,
                 alpha=alpha, gamma=1.5)
    q, k, v = make_inputs(w, DEV)
    run = U.run_prefill(w, q, k, v)
    U.check_against_oracle(w, q, k, v, run, rows=[(0, r, i) for r in range(h_kv) for i in (0, 5, 74, 127, 128, 133, 139, 143, 199)])
