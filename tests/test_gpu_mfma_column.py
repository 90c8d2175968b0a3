"""Layers of one tap and fully connected ones on the matrix cores: filters, channels and positions that fill no tile, a last step
of fewer than 16 channels alone, behind one and behind two others, groups, parts, and what the split cannot carry."""
import sys

import numpy as np
import pytest
import torch

from oracle import spmdm_oracle as so
from paper_1608_01409_amd import binding as B
from paper_1608_01409_amd import workloads as wl

pytestmark = pytest.mark.gpu
TOL = 1e-5

# (C, H, W, K, groups, N): steps of 16 channels and what is left
CONVS = [(15, 40, 40, 32, 1, 30), (17, 40, 40, 32, 1, 30), (32, 19, 23, 65, 1, 30), (33, 9, 11, 65, 1, 80), (41, 31, 7, 97, 1, 60), (96, 28, 28, 70, 2, 33),
         (100, 21, 21, 129, 1, 23), (202, 13, 13, 130, 2, 128), (250, 11, 13, 64, 1, 150)]
FCS = [(100, 512, 1020), (777, 1000, 1020), (2050, 300, 260), (140, 3000, 128)]


@pytest.mark.parametrize("C,H,W,K,groups,N", CONVS)
def test_one_tap(oracle, C, H, W, K, groups, N):
    layer = wl.Layer(f"c{C}k{K}", C, H, W, K, 1, 1, 1, 0, groups)
    rng = np.random.default_rng(C + K)
    w = np.where(rng.random((K, layer.Cg, 1, 1)) < 0.9, rng.standard_normal((K, layer.Cg, 1, 1)) * 0.05, 0).astype(np.float32)
    w[2] = 0
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    print(f"[gpu-case] one tap {layer.name} N={N}", flush=True)
    h = B.sconv_create_csr(layer, w)
    assert B.sconv_route_of(h, N)["kernel"] == "mfma"
    ref, ab, _ = oracle.sparse_conv(layer, w, x)
    xd = torch.from_numpy(x).cuda()
    out = torch.full((N, K, H, W), float("nan"), device="cuda")
    got = B.sconv_forward(h, xd, out).cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= TOL * ab) and np.all(got[ab == 0] == 0)
    bias = rng.standard_normal(K).astype(np.float32) * 0.05
    ref2, scale = oracle.bias_relu(ref, ab, bias, True)
    got = B.sconv_forward_fused(h, xd, torch.from_numpy(bias).cuda(), True).cpu().numpy()
    assert np.all(np.abs(got - ref2) <= TOL * scale)
    # an infinity meets stored weights only, a NaN beyond the last channel of a group nobody
    x[N - 1, layer.Cg - 1, H - 1, W - 1], x[0, C - 1, 0, 0] = np.inf, np.nan
    got = B.sconv_forward(h, torch.from_numpy(x).cuda(), out).cpu().numpy()
    hit = np.zeros(got.shape, bool)
    hit[N - 1, : K // groups, H - 1, W - 1] = w[: K // groups, layer.Cg - 1, 0, 0] != 0
    nan = np.zeros(got.shape, bool)
    nan[0, K - K // groups:, 0, 0] = w[K - K // groups:, layer.Cg - 1, 0, 0] != 0
    assert np.array_equal(np.isinf(got), hit) and np.array_equal(np.isnan(got), nan)
    ok = ~(hit | nan)
    ok[N - 1, :, H - 1, W - 1] = ok[0, :, 0, 0] = False     # (their reference is without the other activation's term)
    assert np.all(np.abs(got[ok].astype(np.float64) - ref[ok]) <= TOL * ab[ok])


@pytest.mark.parametrize("C,K,N", FCS)
def test_fully_connected(C, K, N):
    rng = np.random.default_rng(C + N)
    w = np.where(rng.random((K, C)) < 0.9, rng.standard_normal((K, C)) * 0.05, 0).astype(np.float32)
    x_t = rng.standard_normal((C, N)).astype(np.float32)
    print(f"[gpu-case] column fc C={C} K={K} N={N}", flush=True)
    h = B.sconv_create_csr(B.fc_layer(C, K), w.reshape(K, C, 1, 1))
    assert B.sconv_fc_route_of(h, N)["kernel"] == "mfma"
    ref, ab = so.spmdm(w, x_t)
    out = torch.full((K, N), float("nan"), device="cuda")
    got = B.sconv_fc_forward(h, torch.from_numpy(x_t).cuda(), None, False, out).cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= TOL * ab)


@pytest.mark.parametrize("C,H,W,K,groups,N", [(15, 40, 40, 32, 1, 30), (41, 31, 7, 97, 1, 60), (202, 13, 13, 130, 2, 128)])
def test_activations_that_the_split_cannot_carry(oracle, C, H, W, K, groups, N):
    """Finite activations of 2^111 and more, in the first, the last and one of the middle workgroups."""
    layer = wl.Layer(f"c{C}k{K}", C, H, W, K, 1, 1, 1, 0, groups)
    rng = np.random.default_rng(C * K)
    w = np.where(rng.random((K, layer.Cg, 1, 1)) < 0.9, rng.standard_normal((K, layer.Cg, 1, 1)) * 0.05, 0).astype(np.float32)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    for n, c, y, q in ((0, 0, 0, 0), (N // 2, C // 2, H // 2, 3), (N - 1, C - 1, H - 1, W - 1)):
        x[n, c, y, q] = np.float32(1.7 * 2.0 ** 120)
        x[n, C - 1 - c, y, q] = np.float32(-1.3 * 2.0 ** 111)
    print(f"[gpu-case] one tap, large activations {layer.name} N={N}", flush=True)
    h = B.sconv_create_csr(layer, w)
    assert B.sconv_route_of(h, N)["kernel"] == "mfma"
    ref, ab, _ = oracle.sparse_conv(layer, w, x)
    xd = torch.from_numpy(x).cuda()
    got = B.sconv_forward(h, xd).cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= TOL * ab)
    bias = rng.standard_normal(K).astype(np.float32)
    ref2, scale = oracle.bias_relu(ref, ab, bias, True)
    got = B.sconv_forward_fused(h, xd, torch.from_numpy(bias).cuda(), True).cpu().numpy()
    assert np.all(np.abs(got - ref2) <= TOL * scale)


def relative(got, exact):
    return ((got.double() - exact).square().sum() / exact.square().sum()).sqrt().item()


def exact_and_inputs(layer, N, density, seed):
    """Weights under a mask, rectified activations, a bias, and the sums in 64 bits as [K][N * positions] on the GPU (one group)."""
    rng = np.random.default_rng(seed)
    w = np.where(rng.random((layer.K, layer.C)) < density, rng.standard_normal((layer.K, layer.C)) * 0.05, 0).astype(np.float32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    x = torch.randn((layer.C, N * layer.H * layer.W), generator=gen, device="cuda").clamp_(min=0)
    bias = torch.from_numpy((rng.standard_normal(layer.K) * 0.05).astype(np.float32)).cuda()
    return w, x, bias, torch.from_numpy(w).cuda().double() @ x.double()


# C, H = W, K, N, density: calls that the column kernel takes from the gather kernel of four positions
@pytest.mark.parametrize("C,hw,K,N,density", [(113, 54, 332, 5, 0.2245), (60, 54, 47, 10, 0.6579), (44, 7, 143, 109, 0.7501), (46, 53, 78, 11, 0.4707)])
def test_no_further_from_the_exact_sums_than_the_gather_kernel(C, hw, K, N, density):
    """That kernel's arithmetic step by step: eight products in a chain of 32 bits, the chains and the entries of the first and last channel in 64."""
    layer = wl.Layer("gathered", C, hw, hw, K, 1, 1, 1, 0, 1)
    w, x, bias, exact = exact_and_inputs(layer, N, density, C)
    print(f"[gpu-case] column against gather {C} {hw} {K} {N}", flush=True)
    h = B.sconv_create_csr(layer, w.reshape(K, C, 1, 1))
    assert B.sconv_route_of(h, N)["kernel"] == "mfma" and (w != 0).sum(1).max() <= 48
    sums = torch.zeros_like(exact)
    for k in range(K):
        cols = np.flatnonzero(w[k])
        inner = [c for c in cols if 0 < c < C - 1]
        for i in range(0, len(inner), 8):
            chain = torch.zeros_like(x[0])
            for c in inner[i:i + 8]:
                chain = (x[c].double() * float(w[k, c]) + chain.double()).float()
            sums[k] += chain.double()
        for c in set(cols) - set(inner):
            sums[k] += x[c].double() * float(w[k, c])
    xd = x.view(C, N, hw * hw).transpose(0, 1).reshape(N, C, hw, hw).contiguous()
    rows = lambda t: t.view(N, K, hw * hw).transpose(0, 1).reshape(K, -1)  # noqa: E731
    assert relative(rows(B.sconv_forward(h, xd)), exact) <= relative(sums.float(), exact)
    with_bias = exact + bias.double()[:, None]
    assert relative(rows(B.sconv_forward_fused(h, xd, bias, False)), with_bias) <= relative((sums + bias.double()[:, None]).float(), with_bias)


# C, K, N, density: fully connected calls that it takes from flat streams of 1, 4, 6, 8 and 32 parts; from 12 and 16 in one
@pytest.mark.parametrize("C,K,N,density", [(268, 3276, 480, 0.1558), (210, 3785, 344, 0.5432), (238, 1351, 812, 0.5591), (770, 1513, 144, 0.9151), (2263, 240, 476, 0.4298),
                                         (295, 253, 712, 0.9), (350, 470, 596, 0.407), (402, 491, 720, 0.96)])
def test_no_further_from_the_exact_sums_than_the_flat_streams(C, K, N, density):
    layer = B.fc_layer(C, K)
    w, x, bias, exact = exact_and_inputs(layer, N, density, C)
    print(f"[gpu-case] column against flat streams {C} {K} {N}", flush=True)
    h = B.sconv_create_csr(layer, w.reshape(K, C, 1, 1))
    assert B.sconv_fc_route_of(h, N)["kernel"] == "mfma"
    left = B.sconv_create_csr(layer, w.reshape(K, C, 1, 1), B.sconv_fc_plan(h, N))
    assert B.sconv_fc_route_of(left, N)["kernel"] in ("flat", "flow")
    assert relative(B.sconv_fc_forward(h, x), exact) <= relative(B.sconv_fc_forward(left, x), exact)
    with_bias = exact + bias.double()[:, None]
    assert relative(B.sconv_fc_forward(h, x, bias), with_bias) <= relative(B.sconv_fc_forward(left, x, bias), with_bias)
