"""The forward calls with tensors that the native path declines: what they did on a handle's first call they do on the later ones."""
import numpy as np
import pytest
import torch

from paper_1608_01409_amd import binding as B
from paper_1608_01409_amd import workloads as wl

pytestmark = pytest.mark.gpu


class Sub(torch.Tensor):
    pass


@pytest.mark.parametrize("entry", ["forward", "fused", "noalloc", "fc"])
def test_declined_tensors(entry):
    rng = np.random.default_rng(3)
    layer = B.fc_layer(40, 24) if entry == "fc" else wl.small_layer("calls", C=8, H=6, W=7, K=24, R=3, S=3, pad=1)
    w = np.where(rng.random((24, layer.Cg, layer.R, layer.S)) < 0.4, rng.standard_normal((24, layer.Cg, layer.R, layer.S)), 0).astype(np.float32)
    bias = torch.from_numpy(rng.standard_normal(24).astype(np.float32)).cuda()
    h = B.sconv_create_csr(layer, w)
    shape, out_shape = ((40, 8), (24, 8)) if entry == "fc" else ((4, 8, 6, 7), (4, 24, 6, 7))
    x = torch.randn(shape, device="cuda")

    def call(x, out=None, bias=bias, **kw):
        if out is None:
            out = torch.full(out_shape, float("nan"), device="cuda")
        if entry == "fc":
            return B.sconv_fc_forward(h, x, bias, True, out, **kw)
        if entry == "fused":
            return B.sconv_forward_fused(h, x, bias, True, out, **kw)
        return (B.sconv_forward if entry == "forward" else B.sconv_forward_noalloc)(h, x, out, **kw)

    if entry == "noalloc":
        B.sconv_forward(h, x)
    want = call(x).clone()
    assert want.isfinite().all()
    print(f"[gpu-case] calls {entry}", flush=True)
    given = torch.full(out_shape, float("nan"), device="cuda")
    assert call(x, given) is given and torch.equal(given, want)
    assert torch.equal(call(torch.nn.Parameter(x)), want) and torch.equal(call(x.as_subclass(Sub)), want)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for kw in (dict(stream=side), {}):
        with torch.cuda.stream(side):
            got = call(x, **kw)
        side.synchronize()
        assert torch.equal(got, want)
    # another device, type, shape, order of the dimensions, gaps
    spread = torch.randn(shape + (2,), device="cuda")[..., 0]
    for bad in (x.cpu(), x.double(), x[:, 1:].contiguous(), x[1:].contiguous(), x.transpose(0, 1), spread):
        with pytest.raises(AssertionError):
            call(bad)
    for bad in (given.cpu(), given.double(), given[:, 1:].contiguous(), given.flatten(), given.mT):
        with pytest.raises(AssertionError):
            call(x, bad)
    if entry in ("fused", "fc"):
        for bad in (bias[1:], bias.cpu(), bias.double()):
            with pytest.raises(AssertionError):
                call(x, bias=bad)
    else:
        with pytest.raises(B.SconvError) as e:
            call(x[:0], given[:0])
        assert e.value.status in (B.ERR["NULL"], B.ERR["BATCH"])
    h.destroy()
    with pytest.raises((B.SconvError, AssertionError)):
        call(x)


def native_call(entry):
    """(handle, its input, its output, bias, the native call with the last three, None where it is declined)"""
    rng = np.random.default_rng(4)
    layer = B.fc_layer(40, 24) if entry == "fc" else wl.small_layer("native", C=8, H=6, W=7, K=24, R=3, S=3, pad=1)
    w = np.where(rng.random((24, layer.Cg, layer.R, layer.S)) < 0.4, rng.standard_normal((24, layer.Cg, layer.R, layer.S)), 0).astype(np.float32)
    h = B.sconv_create_csr(layer, w)
    shape, out_shape = ((40, 8), (24, 8)) if entry == "fc" else ((4, 8, 6, 7), (4, 24, 6, 7))
    x, out = torch.randn(shape, device="cuda"), torch.full(out_shape, float("nan"), device="cuda")
    bias = torch.from_numpy(rng.standard_normal(24).astype(np.float32)).cuda()

    def native(x, out, bias):
        f = getattr(B._call, entry)
        return f(h._native, x, bias, True, out) if entry in ("fused", "fc") else f(h._native, x, out)

    return h, x, out, bias, native


def python_lines(entry, h, x, out, bias):
    if entry == "fc":
        return B.sconv_fc_forward(h, x, bias, True, out)
    if entry == "fused":
        return B.sconv_forward_fused(h, x, bias, True, out)
    return (B.sconv_forward if entry == "forward" else B.sconv_forward_noalloc)(h, x, out)


@pytest.mark.parametrize("entry", ["forward", "fused", "noalloc", "fc"])
def test_native_call_takes_plain_tensors_and_no_others(entry):
    h, x, out, bias, native = native_call(entry)
    print(f"[gpu-case] native {entry}", flush=True)
    if entry == "noalloc":
        B.sconv_forward(h, x)
    want = python_lines(entry, h, x, torch.empty_like(out), bias)      # (the first call of a handle)
    assert h._native is not None
    assert native(x, out, bias) == 0 and torch.equal(out, want)
    spread = torch.randn(tuple(x.shape) + (2,), device="cuda")[..., 0]
    assert native(torch.nn.Parameter(x), out, bias) == 0
    for bad in (x.as_subclass(Sub), x.cpu(), x.double(), x[:, 1:].contiguous(), x[1:].contiguous(), x.transpose(0, 1), spread, None):
        assert native(bad, out, bias) is None
    for bad in (None, out.cpu(), out.double(), out[:, 1:].contiguous(), out.flatten(), out.mT):
        assert native(x, bad, bias) is None
    if entry in ("fused", "fc"):
        assert native(x, out, None) == 0
        for bad in (bias[1:], bias.cpu(), bias.double(), bias[:, None], 1.0):
            assert native(x, out, bad) is None


@pytest.mark.parametrize("entry", ["forward", "fused", "noalloc", "fc"])
def test_without_the_native_calls(entry, monkeypatch):
    """What a tree without them does: the same results, from the Python lines."""
    h, x, out, bias, native = native_call(entry)
    print(f"[gpu-case] without native {entry}", flush=True)
    B.sconv_fc_forward(h, x) if entry == "fc" else B.sconv_forward(h, x)
    native(x, out, bias)
    h2 = native_call(entry)[0]
    B._use_torch()
    monkeypatch.setattr(B, "_call", None)
    for _ in range(2):
        if entry == "noalloc":
            B.sconv_forward(h2, x)
        got = python_lines(entry, h2, x, torch.empty_like(out), bias)
        assert h2._native is None and torch.equal(got, out)
