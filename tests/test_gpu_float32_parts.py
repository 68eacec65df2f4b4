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
