"""GPU parity of the forward on both sides of each choice its plan makes from
the grid: the two-group kernel or the 4-wave kernel with 1, 2 or 4 waves per 32
queries, with and without key ranges, and the orders of a causal grid's tiles.
Ragged lengths around the 32-row tiles; the oracle recomputes the first and last
(batch, head) slices.  The bars are those of the other forward tests."""
import pytest
import torch

import oracle
from paper_2112_05682_amd import attention_fwd
from paper_2112_05682_amd.inputs import attention_inputs
from parity_util import TOL, check, check_lse, f64, to_gpu

gpu = pytest.mark.gpu

# (B, H, n_q, n_k, d, d_v, causal): waves per 32 queries and key ranges
GRIDS_16 = [
    (1, 2, 129, 300, 64, 64, True),     # 4 waves, 1 range
    (1, 1, 130, 700, 64, 64, True),     # 4 waves, 2 ranges
    (10, 16, 100, 97, 64, 64, True),    # 2 waves
    (16, 20, 65, 65, 64, 64, True),     # 1 wave, folded order
    (17, 40, 65, 65, 64, 64, True),     # 1 wave, tile-major order (680 workgroups)
    (1, 2, 100, 300, 64, 64, False),    # 4 waves
    (1, 1, 70, 1100, 64, 64, False),    # 4 waves, 5 ranges
    (1, 1, 70, 2500, 64, 64, False),    # 4 waves, 7 ranges
    (13, 10, 65, 2100, 64, 64, False),  # 4 waves
    (13, 10, 65, 130, 64, 64, False),   # 4 waves
    (20, 30, 65, 33, 64, 64, False),    # 1 wave
    (15, 15, 400, 600, 64, 64, False),  # two-group
    (2, 2, 500, 9000, 64, 64, False),   # 4 waves, 8 ranges
    (1, 2, 100, 200, 128, 128, False),  # 2 waves
    (1, 1, 70, 1100, 128, 128, False),  # 2 waves, 6 ranges
    (20, 20, 65, 70, 128, 128, False),  # 1 wave
    (1, 2, 100, 100, 128, 128, True),   # 2 waves
    (1, 1, 1100, 1100, 128, 128, True),  # 2 waves, 2 ranges
    (17, 16, 65, 65, 128, 128, True),   # 1 wave
    (1, 1, 70, 1100, 64, 128, False),   # 2 waves, 6 ranges
    (5, 8, 65, 2100, 128, 64, False),   # 1 wave, 6 ranges
    (17, 16, 65, 70, 64, 128, True),    # 1 wave
]
GRIDS_32 = [
    (1, 1, 70, 300, 64, 64, False),     # 1 wave, 2 ranges
    (5, 8, 65, 600, 64, 64, False),     # 1 wave, 4 ranges
    (5, 8, 129, 129, 64, 64, True),     # 1 wave
    (1, 1, 70, 300, 128, 128, True),    # 2 waves
    (5, 8, 65, 600, 128, 128, False),   # 1 wave, 4 ranges
    (1, 1, 70, 300, 64, 128, False),    # 2 waves, 2 ranges
    (5, 8, 65, 600, 128, 64, False),    # 1 wave, 4 ranges
]
# Grids just past a round, and long causal ones, with the ranges that even them out.
GRIDS_RANGES = [
    (3, 11, 1000, 4100, 64, 64, False),   # two-group, 3 ranges
    (5, 14, 1000, 4100, 64, 64, False),   # two-group, 3 ranges
    (3, 11, 257, 2100, 128, 128, False),  # two-group, 3 ranges
    (1, 1, 65, 9000, 128, 128, False),    # 2 waves, 47 ranges: the staged combine
    (1, 1, 65, 9000, 64, 128, False),     # 2 waves, 47 ranges
    (10, 15, 100, 2100, 128, 64, False),  # 1 wave, 3 ranges
    (1, 2, 3100, 3100, 64, 64, True),     # 1 wave, 13 ranges
    (1, 1, 3100, 3073, 128, 128, True),   # two-group, 13 ranges
    (1, 1, 3100, 3100, 64, 128, True),    # 1 wave, 13 ranges
    (1, 1, 3072, 3072, 128, 64, True),    # 1 wave, 13 ranges
]


def run(shape, dtype, kv_len=None):
    B, H, nq, nk, d, dv, causal = shape
    print("grid case", shape, dtype, kv_len, flush=True)
    x = attention_inputs(B, H, nq, nk, d, dtype, d_v=dv, with_grad=False)
    g = to_gpu(x)
    lens = None if kv_len is None else torch.tensor(kv_len, dtype=torch.int32, device="cuda")
    o, lse = attention_fwd(g["q"], g["k"], g["v"], causal=causal, kv_len=lens)
    torch.cuda.synchronize()
    assert torch.isfinite(o).all()
    for b, h in sorted({(0, 0), (B - 1, H - 1)}):
        sl = tuple(f64(x[t][b:b + 1, h:h + 1]) for t in ("q", "k", "v"))
        ro, rl = oracle.fwd(*sl, scale=d ** -0.5, causal=causal, kv_len=None if kv_len is None else kv_len[b:b + 1])
        check("O", f64(o[b:b + 1, h:h + 1]), ro, TOL[dtype])
        check_lse(f64(lse[b:b + 1, h:h + 1]), rl)


@gpu
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("shape", GRIDS_16, ids=lambda s: "x".join(map(str, s)))
def test_forward_grids_16bit(shape, dtype):
    run(shape, dtype)


@gpu
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("shape", GRIDS_RANGES, ids=lambda s: "x".join(map(str, s)))
def test_forward_grids_with_ranges(shape, dtype):
    run(shape, dtype)


@gpu
@pytest.mark.parametrize("shape", [GRIDS_RANGES[0], GRIDS_RANGES[2], GRIDS_RANGES[6], GRIDS_RANGES[7]],
                         ids=lambda s: "x".join(map(str, s)))
def test_grids_with_ranges_and_padding(shape):
    # Valid lengths that leave the later ranges without a key.
    run(shape, "bf16", kv_len=[200 + 700 * b for b in range(shape[0])])


@gpu
@pytest.mark.parametrize("shape", GRIDS_32, ids=lambda s: "x".join(map(str, s)))
def test_forward_grids_float32(shape):
    run(shape, "fp32")


@gpu
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("fp32", 64), ("fp32", 128)])
@pytest.mark.parametrize("causal", [False, True])
def test_forward_shared_queries_with_padding(dtype, d, causal):
    # Valid lengths inside, at and past a wave's 32 keys of the staged tile:
    # some waves, and some key ranges, see no key at all.
    run((5, 1, 70, 600, d, d, causal), dtype, kv_len=[1, 31, 64, 97, 600])


@gpu
@pytest.mark.parametrize("d", [64, 128])
def test_rows_without_keys(d):
    # A batch without valid keys: o = 0 and lse = -inf through the waves' combine.
    g = to_gpu(attention_inputs(2, 1, 70, 100, d, "bf16", with_grad=False))
    lens = torch.tensor([0, 100], dtype=torch.int32, device="cuda")
    o, lse = attention_fwd(g["q"], g["k"], g["v"], kv_len=lens)
    assert (o[0] == 0).all() and (lse[0] == -float("inf")).all() and torch.isfinite(lse[1]).all()


@gpu
@pytest.mark.parametrize("dtype,d,first", [("bf16", 64, 32), ("bf16", 64, 96), ("bf16", 128, 32), ("fp32", 64, 32),
                                           ("fp32", 128, 32)])
def test_nan_scores_of_one_wave(dtype, d, first):
    # Keys that one of the waves sharing a tile's queries has for itself, all NaN:
    # o is NaN and lse -inf, as where one wave sees them beside other keys.
    n = first + 7
    g = to_gpu(attention_inputs(1, 1, 70, n, d, dtype, with_grad=False))
    for i in (first, 3):
        k = g["k"].clone()
        k[0, 0, i:n if i == first else i + 1] = float("nan")
        o, lse = attention_fwd(g["q"], k, g["v"])
        assert o.isnan().all() and (lse == -float("inf")).all()


@gpu
@pytest.mark.parametrize("shape", [
    (8, 13, 330, 330, 64, 64),    # 1 wave, folded (312 workgroups of 3 tiles a head)
    (7, 8, 330, 257, 128, 128),   # 2 waves, folded (336 of 6)
    (8, 25, 330, 330, 64, 64),    # 1 wave, tile major (600)
    (7, 25, 270, 270, 128, 128),  # 1 wave, tile major (525)
    (8, 8, 600, 600, 64, 128),    # 1 wave, folded (320 of 5)
], ids=lambda s: "x".join(map(str, s)))
def test_causal_orders_every_slice(shape):
    # Grids of more than 256 workgroups and several tiles a head: every slice.
    B, H, nq, nk, d, dv = shape
    x = attention_inputs(B, H, nq, nk, d, "bf16", d_v=dv, with_grad=False)
    g = to_gpu(x)
    o, lse = attention_fwd(g["q"], g["k"], g["v"], causal=True)
    ro, rl = oracle.fwd(*(f64(x[t]) for t in ("q", "k", "v")), scale=d ** -0.5, causal=True)
    check("O", f64(o), ro, TOL["bf16"])
    check_lse(f64(lse), rl)


def test_tile_orders_cover_every_item_once():
    """The three orders of causal_tile_order (tile_item in device.hpp), restated:
    each maps the workgroups of a grid to its (tile, group) items one to one."""
    def item(w, n, n_tiles, order):
        if order == 0:
            x, i = w & 7, w >> 3
            per, rem = n >> 3, n & 7
            g = x * per + min(x, rem) + i
            return g % n_tiles, g // n_tiles
        x, i = w & 7, w >> 3
        n_x, r0 = (n - x + 7) >> 3, i & ~31
        cnt = min(n_x - r0, 32)
        j = r0 + cnt - 1 - (i - r0) if order == 2 and r0 & 32 else i
        g, groups = 8 * j + x, n // n_tiles
        return g // groups, g % groups

    for n_tiles, groups in ((1, 1), (3, 7), (16, 32), (5, 101), (9, 57), (511, 1), (8, 64)):
        n = n_tiles * groups
        for order in (0, 1, 2):
            items = {item(w, n, n_tiles, order) for w in range(n)}
            assert items == {(t, g) for t in range(n_tiles) for g in range(groups)}
