"""A NaN or an infinity in one token reaches what attends that token and nothing else: the fp32
kernels walk the chunk lists of 16 rows together, and a weight of 0 times a NaN is a NaN."""
import pytest
import torch

import parity_util as U
from paper_2605_18753_amd import binding as B
from paper_2605_18753_amd.inputs import Workload, make_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# heads per group, tokens, head dimension, chunk, causal: ragged row tiles, one and several parts per list
SHAPES = [(4, 333, 128, 64, True), (1, 257, 64, 64, True), (16, 130, 64, 64, True), (2, 640, 64, 128, False),
          (1, 1100, 128, 64, True)]


def setup(g, n, d, block, causal):
    w = Workload("nonfinite", 1, 2 * g, 2, n, n, d, block, causal=causal, dtype="fp32", offset_sigma=1.0, gamma=3.0, seed=51)
    q, k, v = (t.to(DEV) for t in make_inputs(w, "cpu"))
    run = U.run_prefill(w, q, k, v)
    bits = torch.stack([(run.lists.mask[0, 0, :, c // 32] >> (c % 32)) & 1 for c in range(B.list_stride(run.params))], 1).bool()
    # att[i, j]: token i of kv-head 0 attends key j
    key = torch.arange(n, device=DEV)
    att = bits[:, key // block]
    if causal:
        att &= key[None, :] <= key[:, None]
    return w, q, k, v, run, att


def poisoned(t, head, row, value):
    t = t.clone()
    t[0, head, row] = value
    return t


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_forward_rows_that_do_not_attend_the_key_are_untouched(shape, value):
    g, n, d, block, causal = shape
    w, q, k, v, run, att = setup(*shape)
    ws = B.alloc_workspace(run.params, DEV)
    dense = torch.empty_like(q)
    B.dense_attn(run.params, q, k, v, dense, ws)
    for j in (n // 3, n - 3):
        for which in ("k", "v"):
            kk, vv = (poisoned(k, 0, j, value), v) if which == "k" else (k, poisoned(v, 0, j, value))
            for clean_o, is_dense in ((run.o, False), (dense, True)):
                o = torch.empty_like(q)
                if is_dense:
                    B.dense_attn(run.params, q, kk, vv, o, ws)
                    hit = torch.arange(n, device=DEV) >= j if causal else torch.ones(n, dtype=torch.bool, device=DEV)
                else:
                    B.dash_stage2_attend(run.params, q, kk, vv, o, run.lists, ws)
                    hit = att[:, j]
                torch.cuda.synchronize()
                assert hit.any() and (is_dense or not hit.all())
                assert torch.equal(o[0, g:], clean_o[0, g:])                      # the other kv-head
                same = torch.equal(o[0, :g][:, ~hit], clean_o[0, :g][:, ~hit])
                assert same, (which, j, is_dense)
                if which == "v" or value != value:
                    reached = not bool(torch.isfinite(o[0, :g][:, hit]).any())
                    assert reached, (which, j, is_dense)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("which", ["q", "k", "v", "d_o"])
def test_backward_of_what_does_not_meet_the_token_is_untouched(shape, which):
    g, n, d, block, causal = shape
    w, q, k, v, run, att = setup(*shape)
    d_o = torch.randn(q.shape, generator=torch.Generator().manual_seed(52)).to(DEV)
    wsb = B.alloc_backward_workspace(run.params, DEV)

    def grads(q, k, v, d_o):
        out = [torch.full_like(t, 7.0) for t in (q, k, v)]
        B.dash_attn_backward(run.params, q, k, v, d_o, run.kbar, run.lists, *out, wsb)
        torch.cuda.synchronize()
        return out

    clean = grads(q, k, v, d_o)
    for tok in (n - 3, n // 2 + 1):
        t = dict(q=q, k=k, v=v, d_o=d_o)
        t[which] = poisoned(t[which], 0, tok, float("nan"))      # head 0 of kv-head 0's group
        got = grads(**t)
        # tokens whose weights or upstream gradient are NaN (all heads of the group count as one)
        rows = att[:, tok].clone() if which in "kv" else torch.arange(n, device=DEV) == tok
        keys_v = att[rows].any(0)
        # dk: the attended keys, and all keys of the chunks a hit token routed to (through their summaries)
        chunk = torch.arange(n, device=DEV) // block
        own = torch.arange(n, device=DEV)[:, None] // block == chunk[None, :]
        routed = (att & ~own if causal else att)[rows].any(0)
        if n % block:
            routed &= chunk < n // block
        keys_k = keys_v | routed
        assert not rows.all()
        for name, a, b, hit, heads in (("dq", got[0], clean[0], rows, g), ("dk", got[1], clean[1], keys_k, 1), ("dv", got[2], clean[2], keys_v, 1)):
            far = a[0, :heads][:, ~hit]
            bad = int((~torch.isfinite(far)).sum()) + int((~torch.isfinite(a[0, heads:])).sum())     # ... and the other kv-head
            assert bad == 0, (name, tok)
            # parts of a list are added in no fixed order: a few roundings of the largest element
            assert (far - b[0, :heads][:, ~hit]).abs().max() <= 1e-6 * b.abs().max() if far.numel() else True, name
        # and it does reach what meets it
        reached = not bool(torch.isfinite(got[0][0, 0, rows]).any())
        assert reached


@pytest.mark.parametrize("dtype,g,n,d,block", [("bf16", 4, 333, 128, 64), ("bf16", 2, 129, 64, 64), ("bf16", 16, 195, 128, 128),
                                               ("bf16", 1, 1000, 64, 64), ("fp32", 4, 333, 128, 64)])
def test_rows_behind_the_end_of_a_padded_buffer_are_not_used(dtype, g, n, d, block):
    w = Workload("padded", 2, 2 * g, 2, n, n, d, block, dtype=dtype, offset_sigma=0.8, gamma=2.0, seed=53)
    q, k, v = (t.to(DEV) for t in make_inputs(w, "cpu"))
    d_o = torch.randn(q.shape, generator=torch.Generator().manual_seed(54)).to(q.dtype).to(DEV)

    def step(q, k, v, d_o):
        # o and d_o share their strides
        o = torch.empty(d_o.untyped_storage().nbytes() // d_o.element_size(), dtype=q.dtype, device=DEV).as_strided(d_o.shape, d_o.stride())
        p = B.make_params(q, k, v, o, block, w.alpha, w.gamma, w.sigma, True)
        kbar = torch.empty(B.kbar_shape(p), dtype=torch.float32, device=DEV)
        lists = B.Lists.allocate(p, DEV)
        B.dash_attn_prefill(p, q, k, v, o, kbar, lists, B.alloc_workspace(p, DEV))
        out = [torch.empty_strided(t.size(), t.stride(), dtype=t.dtype, device=DEV) for t in (q, k, v)]
        B.dash_attn_backward(p, q, k, v, d_o, kbar, lists, *out, B.alloc_backward_workspace(p, DEV))
        torch.cuda.synchronize()
        return [o] + out

    def padded(t):
        big = torch.full((t.shape[0], t.shape[1], n + 40, d), float("nan"), dtype=t.dtype, device=DEV)
        big[:, :, :n] = t
        return big[:, :, :n]

    for name, a, b in zip(("o", "dq", "dk", "dv"), step(*(padded(t) for t in (q, k, v, d_o))), step(q, k, v, d_o)):
        bad = int((~torch.isfinite(a.float())).sum())
        assert bad == 0, name
        # fp32: parts of a list are added in no fixed order
        same = torch.equal(a, b) if dtype == "bf16" else bool((a - b).abs().max() <= 1e-6 * b.abs().max())
        assert same, name
