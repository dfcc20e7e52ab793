"""The exponentials of the fp32 attention: one rounding of e^x, not of its argument in base 2."""
import pytest
import torch

from paper_2605_18753_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("d", [64, 128])
def test_attention_weights_to_one_ulp(d):
    """K = V = the identity makes the output the weights themselves, of logits that are multiples of 2^-9 in
    [-20, 0], so that scores and differences are exact and all weights stay normal numbers.  A weight over its row's
    largest (whose exponential is exactly 1) then carries e^x to 1 ulp (2^-23), and half an ulp from the
    normalisation of each of the two: 2^-22 = 2.4e-7.  A rounded product x log2(e) alone is off by 2^-25 |x log2(e)| ln 2
    units: up to 6.6e-7 here."""
    n = 64
    gen = torch.Generator().manual_seed(61)
    z = -torch.randint(0, 20 * 512 + 1, (n, n), generator=gen).double() / 512
    q = torch.zeros(1, 1, n, d)
    q[0, 0, :, :n] = z.float()
    eye = torch.zeros(1, 1, n, d)
    eye[0, 0, :, :n] = torch.eye(n)
    q, k = q.to(DEV), eye.to(DEV)
    o = torch.empty_like(q)
    p = B.make_params(q, k, k, o, 64, causal=False, scale=1.0)
    B.dense_attn(p, q, k, k, o, B.alloc_workspace(p, DEV))
    torch.cuda.synchronize()
    w = o[0, 0, :, :n].double().cpu()
    top = z.argmax(1, keepdim=True)
    want = torch.exp(z - z.gather(1, top))
    err = ((w / w.gather(1, top)) / want - 1).abs()
    print(f"worst {err.max():.2e} rms {err.square().mean().sqrt():.2e}")
    assert float(err.max()) <= 2.0 ** -22 * 1.01          # 1 %: the products of the three roundings
