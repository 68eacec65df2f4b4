"""float32 operands are summed from three bf16 parts each: values that have
fewer bits to spare than ordinary ones.  Powers of two scale every part
exactly, so they must come through bitwise; infinities and the largest finite
values must not turn into NaN where float32 products would not."""
import pytest
import torch

from paper_2112_05682_amd import attention_bwd, attention_fwd
from paper_2112_05682_amd.inputs import attention_inputs
from parity_util import to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,dv", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("causal", [False, True])
def test_powers_of_two_scale_exactly(d, dv, causal):
    x = to_gpu(attention_inputs(1, 2, 70, 133, d, "fp32", d_v=dv))
    o, lse = attention_fwd(x["q"], x["k"], x["v"], causal=causal)
    grads = attention_bwd(x["q"], x["k"], x["v"], o, lse, x["do"], causal=causal)
    for e in (-60, 100):  # parts of 2^-60 values end near 2^-84, far above the smallest bf16
        s = 2.0 ** e
        o2, lse2 = attention_fwd(x["q"], x["k"], x["v"] * s, causal=causal)
        assert torch.equal(o2, o * s) and torch.equal(lse2, lse)
    for e in (-40, 40):
        s = 2.0 ** e
        for a, b in zip(attention_bwd(x["q"], x["k"], x["v"], o, lse, x["do"] * s, causal=causal), grads):
            assert torch.equal(a, b * s)


@pytest.mark.parametrize("d", [64, 128])
def test_infinite_and_largest_values_pass(d):
    x = to_gpu(attention_inputs(1, 1, 40, 70, d, "fp32"))
    v = x["v"].clone()
    v[0, 0, 5, 3] = float("inf")
    v[0, 0, 6, 4] = -float("inf")
    v[0, 0, 7, 5] = float("nan")
    o, _ = attention_fwd(x["q"], x["k"], v)
    assert (o[..., 3] == float("inf")).all() and (o[..., 4] == -float("inf")).all() and o[..., 5].isnan().all()
    rest = [f for f in range(d) if f not in (3, 4, 5)]
    assert torch.equal(o[..., rest], attention_fwd(x["q"], x["k"], x["v"])[0][..., rest])
    # One key: o is v, also above the largest bf16, up to the rounding of the
    # weight, the product, the reciprocal and its product (2^-24 each).
    big = torch.full((1, 1, 1, d), 0.999 * torch.finfo(torch.float32).max, device="cuda")
    o, _ = attention_fwd(x["q"], x["k"][:, :, :1], big)
    assert ((o / big - 1).abs() <= 2.0 ** -22).all()


def rel(a, b):
    """2-norm of the difference over that of b, in float64."""
    return float((a.double() - b).norm() / b.norm())


@pytest.mark.parametrize("d,dv", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("n_q,n_k,causal", [(70, 133, False), (70, 70, True), (140, 600, False)])
def test_smallest_values_keep_their_bits(d, dv, n_q, n_k, causal):
    """Values of 2^-118 times N(0, 1), whose bf16 parts would end below the smallest
    bf16 (2^-133): a few bits would be missing, 8e-6 and more of the results.  In
    float32 itself the smallest numbers here are the dS = P dP near 2^-118 / n_k:
    at 600 keys 2^-127, which round to multiples of 2^-149, half of that or 2^-23
    of them each at random, and o's terms likewise: 2^-22 of a result at most."""
    x = to_gpu(attention_inputs(1, 2, n_q, n_k, d, "fp32", d_v=dv))
    s = 2.0 ** -118
    o, lse = attention_fwd(x["q"], x["k"], x["v"], causal=causal)
    g = attention_bwd(x["q"], x["k"], x["v"], o, lse, x["do"], causal=causal)
    o2, lse2 = attention_fwd(x["q"], x["k"], x["v"] * s, causal=causal)
    assert torch.equal(lse2, lse) and rel(o2, o.double() * s) <= 2.0 ** -22
    for a, b in zip(attention_bwd(x["q"], x["k"], x["v"], o, lse, x["do"] * s, causal=causal), g):
        assert rel(a, b.double() * s) <= 2.0 ** -22
    # dS as small as that: v large again.
    for a, b, e in zip(attention_bwd(x["q"], x["k"], x["v"] * s, o2, lse, x["do"], causal=causal), g, (s, s, 1.0)):
        assert rel(a, b.double() * e) <= 2.0 ** -22


@pytest.mark.parametrize("d,dv", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("which", ["q", "k", "v", "do"])
def test_tiles_with_large_values(d, dv, which):
    """Values above 2^18 in one head, which make its tiles start again: powers of
    two scale its results exactly, and the other head's stay as they were."""
    x = to_gpu(attention_inputs(1, 2, 140, 200, d, "fp32", d_v=dv))
    big = torch.tensor([1.0, 2.0 ** 24], device="cuda").view(1, 2, 1, 1)
    back = {"q": "k", "k": "q"}.get(which)  # q k stays what it was
    y = dict(x)
    y[which] = x[which] * big
    if back:
        y[back] = x[back] / big
    o, lse = attention_fwd(x["q"], x["k"], x["v"])
    dq, dk, dv_ = attention_bwd(x["q"], x["k"], x["v"], o, lse, x["do"])
    o2, lse2 = attention_fwd(y["q"], y["k"], y["v"])
    g2 = attention_bwd(y["q"], y["k"], y["v"], o2, lse2, y["do"])
    one = torch.ones_like(big)
    so, sq, sk, sv = {"q": (one, 1 / big, big, one), "k": (one, big, 1 / big, one),
                      "v": (big, big, big, one), "do": (one, big, big, big)}[which]
    assert torch.equal(lse2, lse) and torch.equal(o2, o * so)
    for a, b, s in zip(g2, (dq, dk, dv_), (sq, sk, sv)):
        assert torch.equal(a, b * s)


def test_scales_of_any_size():
    """score_scale 2^-100 and 2^100 with q scaled to match: the same scores."""
    x = to_gpu(attention_inputs(1, 2, 70, 133, 64, "fp32"))
    o, lse = attention_fwd(x["q"], x["k"], x["v"], scale=0.125)
    g = attention_bwd(x["q"], x["k"], x["v"], o, lse, x["do"], scale=0.125)
    for e in (100, -100):
        s = 2.0 ** e
        o2, lse2 = attention_fwd(x["q"] * s, x["k"], x["v"], scale=0.125 / s)
        assert torch.equal(o2, o) and torch.equal(lse2, lse)
        g2 = attention_bwd(x["q"] * s, x["k"], x["v"], o2, lse2, x["do"], scale=0.125 / s)
        for a, b, f in zip(g2, g, (1 / s, 1.0, 1.0)):
            assert torch.equal(a, b * f)


def test_lone_products_round_like_float32():
    """One feature and one key: the log-sum-exp is the product, times the scale,
    log2(e) and ln(2), four roundings at most: 0.64 units of 2^-24 rms (the first
    products after the small ones in one MFMA sum: 0.75)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    q, k = (torch.zeros(1, 4096, 1, 64, device="cuda") for _ in range(2))
    for t in (q, k):
        t[..., 3] = 1 + torch.rand(1, 4096, 1, generator=g, device="cuda")
    _, lse = attention_fwd(q, k, k, scale=1.0)
    s = (q.double() * k.double()).sum(-1)
    e = ((lse.double() - s) / s).abs() * 2.0 ** 24
    assert float(e.square().mean().sqrt()) <= 0.68 and float(e.max()) <= 2.5
