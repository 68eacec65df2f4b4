"""The native marshalling of plain GPU tensors against the general Python path
(the same library underneath): the same bits for every layout, option and
output form that the native calls accept, and None for what they leave to the
general path."""
import ctypes

import pytest
import torch

from paper_2112_05682_amd import (_lib, attention, attention_bwd, attention_fwd, attention_packed)

pytestmark = pytest.mark.gpu


class _Off:
    """Native calls that accept nothing."""

    fwd = bwd = packed_fwd = packed_bwd = staticmethod(lambda *a: None)


def randn(*shape, dtype, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda").to(dtype)


def tensors(layout, dtype, d, dv):
    B, H, nq, nk = 2, 3, 70, 45
    if layout == "bnhd":  # the paper's order, as [B, H, n, d] views
        q, k, v, do = (randn(B, n, H, w, dtype=dtype, seed=i).transpose(1, 2)
                       for i, (n, w) in enumerate(((nq, d), (nk, d), (nk, dv), (nq, dv))))
    elif layout == "shared":  # one key head for every query head
        q, do = randn(B, H, nq, d, dtype=dtype, seed=0), randn(B, H, nq, dv, dtype=dtype, seed=3)
        k, v = (randn(B, 1, nk, w, dtype=dtype, seed=s).expand(B, H, nk, w) for s, w in ((1, d), (2, dv)))
    elif layout == "sliced":  # a column range of wider rows
        q, k, v, do = (randn(B, H, n, w + 32, dtype=dtype, seed=i)[..., 16:16 + w]
                       for i, (n, w) in enumerate(((nq, d), (nk, d), (nk, dv), (nq, dv))))
    else:
        q, k, v, do = (randn(B, H, n, w, dtype=dtype, seed=i)
                       for i, (n, w) in enumerate(((nq, d), (nk, d), (nk, dv), (nq, dv))))
    return q, k, v, do


def both(monkeypatch, f):
    assert _lib.native() is not None
    a = f()
    with monkeypatch.context() as m:
        m.setattr(_lib, "_native", _Off)
        b = f()
    torch.cuda.synchronize()
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert (x is None) == (y is None)
        if x is not None:
            assert x.dtype == y.dtype and x.shape == y.shape and x.stride() == y.stride()
            assert torch.equal(x, y)
    return a


@pytest.mark.parametrize("layout", ["contiguous", "bnhd", "shared", "sliced"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("d,dv", [(64, 64), (64, 128), (128, 128)])
def test_native_calls_match_the_general_path(layout, dtype, d, dv, monkeypatch):
    q, k, v, do = tensors(layout, dtype, d, dv)
    lens = torch.tensor([45, 7], dtype=torch.int32, device="cuda")
    for causal, scale, kv_len, out_dtype in ((False, None, None, None), (True, 0.3, lens, None),
                                             (False, 1, None, torch.float32)):
        native = _lib.native().fwd(q, k, v, causal, scale, True, None, out_dtype, kv_len, True)
        assert native is not None
        o, lse, o_lo = both(monkeypatch, lambda: attention_fwd(q, k, v, causal, scale, out_dtype=out_dtype,
                                                               kv_len=kv_len, residual=True))
        out = torch.empty(2, 70, 3, dv, dtype=o.dtype, device="cuda").transpose(1, 2)
        both(monkeypatch, lambda: attention_fwd(q, k, v, causal, scale, need_lse=False, out=out, kv_len=kv_len,
                                                out_dtype=out_dtype))
        assert attention_fwd(q, k, v, out=out, out_dtype=out_dtype)[0] is out
        g = do.to(o.dtype)
        for need in ((True, True), (True, False), (False, True)):
            both(monkeypatch, lambda: attention_bwd(q, k, v, o, lse, g, causal, scale, *need, kv_len=kv_len,
                                                    o_lo=o_lo))
        given = (torch.empty(2, 70, 3, d, dtype=dtype, device="cuda").transpose(1, 2), None, None)
        both(monkeypatch, lambda: attention_bwd(q, k, v, o, lse, g, causal, scale, out=given, kv_len=kv_len))

    def train():
        x = [t.detach().requires_grad_() for t in (q, k, v)]
        r = attention(*x, causal=True, kv_len=lens)
        return (r, *torch.autograd.grad(r, x, do))

    both(monkeypatch, train)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d", [64, 128])
def test_native_packed_calls_match_the_general_path(dtype, d, monkeypatch):
    qkv = randn(2, 50, 3, 3, d, dtype=dtype, seed=4).requires_grad_()
    lens = torch.tensor([11, 50], dtype=torch.int32, device="cuda")
    for do in (randn(2, 50, 3, d, dtype=dtype, seed=5), randn(2, 3, 50, d, dtype=dtype, seed=5).transpose(1, 2),
               randn(2, 50, 1, d, dtype=dtype, seed=5).expand(2, 50, 3, d)):
        for kv_len in (None, lens):
            def f():
                o = attention_packed(qkv, causal=True, scale=0.2, kv_len=kv_len)
                return o, torch.autograd.grad(o, qkv, do)[0]

            both(monkeypatch, f)


def test_native_calls_leave_other_inputs_to_the_general_path():
    n = _lib.native()
    q, k, v, do = tensors("contiguous", torch.bfloat16, 64, 64)
    for bad in ((q.cpu(), k, v), (q, k.float(), v), (q, k[:, :2], v), (q[0], k[0], v[0]), (q, k, v[:, :, :9]),
                (q.transpose(2, 3), k, v), (q[..., :60], k[..., :60], v)):
        assert n.fwd(*bad, False, None, True, None, None, None, False) is None
    assert n.fwd(q, k, v, False, "x", True, None, None, None, False) is None
    assert n.fwd(q, k, v, False, 0.0, True, None, None, None, False) is None
    assert n.fwd(q, k, v, False, None, True, None, torch.float16, None, False) is None
    assert n.fwd(q, k, v, False, None, True, None, None, torch.zeros(2, device="cuda"), False) is None
    assert n.packed_fwd(q, False, None, None) is None
    o, lse, o_lo = attention_fwd(q, k, v, residual=True)
    assert n.bwd(q, k, v, o, lse, do, False, None, False, False, None, None, o_lo) is None
    assert n.bwd(q, k, v, o, lse, do.float(), False, None, True, True, None, None, o_lo) is None
    assert n.bwd(q, k, v, o, lse[:, :, :5], do, False, None, True, True, None, None, o_lo) is None


@pytest.mark.parametrize("status,raised", [(_lib.MEA_ERR_HIP, True), (_lib.MEA_ERR_WORKSPACE, True),
                                           (_lib.MEA_ERR_INVALID_ARG, False), (_lib.MEA_ERR_UNSUPPORTED, False)])
def test_failed_launches_are_raised_and_not_repeated(status, raised):
    """A library whose launches fail (stand-ins on the host): the native calls raise
    the status, and return None for what the library refuses before a launch."""
    n, lib, calls = _lib.native(), _lib.load(), []
    real = [ctypes.cast(getattr(lib, name), ctypes.c_void_p).value for name in _lib.NATIVE_CALLS]
    stand_in = ctypes.CFUNCTYPE(ctypes.c_int)(lambda: calls.append(1) or status)
    fake = ctypes.cast(stand_in, ctypes.c_void_p).value
    q, k, v, do = tensors("contiguous", torch.bfloat16, 64, 64)
    qkv, dqkv = (randn(2, 50, w, 3, 64, dtype=torch.bfloat16, seed=4) for w in (3, 1))
    o, lse, o_lo = attention_fwd(q, k, v, residual=True)
    po, plse, po_lo = n.packed_fwd(qkv, False, None, None)
    every = [lambda: n.fwd(q, k, v, False, None, True, None, None, None, True),
             lambda: n.bwd(q, k, v, o, lse, do, False, None, True, True, None, None, o_lo),
             lambda: n.packed_fwd(qkv, False, None, None),
             lambda: n.packed_bwd(qkv, po, plse, po_lo, dqkv[:, :, 0], False, None, None)]
    n.init(_lib.check, *real[:2], fake, fake)
    try:
        for f in every:
            if raised:
                with pytest.raises(_lib.MeaError) as e:
                    f()
                assert e.value.status == status
            else:
                assert f() is None
        if raised:  # through the public calls: once, and no second attempt
            with pytest.raises(_lib.MeaError):
                attention_fwd(q, k, v)
            with pytest.raises(_lib.MeaError):
                attention_bwd(q, k, v, o, lse, do)
        assert len(calls) == (6 if raised else 4)
    finally:
        n.init(_lib.check, *real)
    assert torch.equal(attention_fwd(q, k, v)[0], o)
