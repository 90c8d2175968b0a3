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
