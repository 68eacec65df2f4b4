"""GPU parity of the backward on both sides of each choice its launch makes from
the grid: how many waves share a 32-row column (4, 2 or 1), dK/dV and dQ in one
launch or two, and the two-group kernels on grids that fill the chip.  Ragged
lengths around the 32-row tiles; the oracle recomputes the first and last
(batch, head) slices.  The bars are those of the other backward tests."""
import pytest
import torch

import oracle
from paper_2112_05682_amd import attention_bwd, attention_fwd
from paper_2112_05682_amd.inputs import attention_inputs
from parity_util import TOL, check, f64, gradient_row_scales, to_gpu

pytestmark = pytest.mark.gpu

# (B, H, n_q, n_k, d, d_v): waves per column and launches at these sizes
GRIDS = [
    (1, 2, 33, 161, 64, 64),        # four waves per column (at most 128 tiles of 128 rows)
    (1, 1, 129, 31, 64, 64),
    (7, 10, 97, 65, 64, 64),        # two (140 tiles)
    (16, 10, 129, 97, 64, 64),      # one, in one launch (480)
    (1, 2, 33, 161, 128, 128),      # two (at most 128)
    (1, 2, 65, 129, 128, 64),
    (1, 2, 65, 129, 64, 128),
    (16, 5, 129, 97, 128, 128),     # one, in one launch (240)
    (16, 5, 129, 97, 128, 64),
]
# Unmasked 16-bit, keys for more than twice the queries (1.5 times at d = d_v = 128):
# dQ's workgroups before dK/dV's in one launch.
LONG_KEYS = [
    (1, 2, 33, 67, 64, 64),         # four waves per column
    (7, 10, 65, 131, 64, 64),       # two
    (10, 10, 65, 257, 64, 64),      # one
    (10, 10, 65, 98, 128, 128),
    (10, 10, 65, 257, 128, 64),
    (10, 10, 65, 257, 64, 128),
    (3, 1, 70, 6200, 128, 128),     # one, in two launches (3 dQ workgroups)
]
LARGE = [
    ((32, 33, 129, 129, 128, 128), False),  # one, in two launches (4224 tiles)
    ((5, 8, 1030, 1025, 64, 64), False),    # two-group kernels (200 workgroups a pass)
    ((8, 8, 2049, 2050, 64, 64), True),     # two-group kernels, causal (576)
    ((8, 8, 1000, 4100, 64, 64), False),    # two-group kernels, a full round of 256 dQ workgroups
    ((9, 7, 769, 4096, 64, 64), False),     # two-group kernels, 252 of 256
]


def run(shape, dtype, causal, kv_len=None):
    B, H, nq, nk, d, dv = shape
    print("grid case", shape, dtype, causal, kv_len, flush=True)
    x = attention_inputs(B, H, nq, nk, d, dtype, d_v=dv)
    g = to_gpu(x)
    lens = None if kv_len is None else torch.tensor(kv_len, dtype=torch.int32, device="cuda")
    o, lse, o_lo = attention_fwd(g["q"], g["k"], g["v"], causal=causal, kv_len=lens, residual=True)
    args = (g["q"], g["k"], g["v"], o, lse, g["do"], causal)
    both = attention_bwd(*args, kv_len=lens, o_lo=o_lo)
    # A pass that runs alone takes the same shares: the same bits.
    dq, _, _ = attention_bwd(*args, kv_len=lens, o_lo=o_lo, need_dkdv=False)
    _, dk, dv_ = attention_bwd(*args, kv_len=lens, o_lo=o_lo, need_dq=False)
    for name, a, b in zip(("dq", "dk", "dv"), (dq, dk, dv_), both):
        assert torch.equal(a, b), name
    for b, h in sorted({(0, 0), (B - 1, H - 1)}):
        sl = tuple(f64(x[t][b:b + 1, h:h + 1]) for t in ("q", "k", "v", "do"))
        kl = None if kv_len is None else kv_len[b:b + 1]
        ref = oracle.bwd(*sl, scale=d ** -0.5, causal=causal, kv_len=kl)
        _, rl = oracle.fwd(*sl[:3], scale=d ** -0.5, causal=causal, kv_len=kl)
        cq, ck = gradient_row_scales(*sl, rl, d ** -0.5, causal, kv_len=kl)
        for name, got, want, terms in zip(("dQ", "dK", "dV"), both, ref, (cq, ck, None)):
            check(name, f64(got[b:b + 1, h:h + 1]), want, TOL[dtype], terms=terms)


@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("shape", GRIDS, ids=lambda s: "x".join(map(str, s)))
def test_backward_shares_of_a_column(shape, causal, dtype):
    run(shape, dtype, causal)


@pytest.mark.parametrize("shape,causal", LARGE, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else "")
def test_backward_large_grids(shape, causal):
    run(shape, "bf16", causal)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
def test_backward_shared_columns_with_padding(d, causal):
    # Valid lengths inside, at and past a 32-key share of the staged tile.
    run((5, 1, 70, 129, d, d), "bf16", causal, kv_len=[1, 31, 64, 97, 129])


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("shape", LONG_KEYS, ids=lambda s: "x".join(map(str, s)))
def test_backward_grids_long_keys(shape, dtype):
    run(shape, dtype, False)


@pytest.mark.parametrize("shape", [
    (8, 13, 330, 330, 64, 64),    # one launch, resident: dQ's lightest tiles first (624 workgroups)
    (8, 7, 330, 257, 128, 128),   # one launch, 336
    (8, 25, 330, 330, 64, 64),    # one launch, several rounds
], ids=lambda s: "x".join(map(str, s)))
def test_causal_orders_every_slice(shape):
    # Grids of more than 256 workgroups and several tiles a head: every slice.
    B, H, nq, nk, d, dv = shape
    x = attention_inputs(B, H, nq, nk, d, "bf16", d_v=dv)
    g = to_gpu(x)
    o, lse, o_lo = attention_fwd(g["q"], g["k"], g["v"], causal=True, residual=True)
    got = attention_bwd(g["q"], g["k"], g["v"], o, lse, g["do"], True, o_lo=o_lo)
    sl = tuple(f64(x[t]) for t in ("q", "k", "v", "do"))
    ref = oracle.bwd(*sl, scale=d ** -0.5, causal=True)
    _, rl = oracle.fwd(*sl[:3], scale=d ** -0.5, causal=True)
    cq, ck = gradient_row_scales(*sl, rl, d ** -0.5, True)
    for name, a, want, terms in zip(("dQ", "dK", "dV"), got, ref, (cq, ck, None)):
        check(name, f64(a), want, TOL["bf16"], terms=terms)
