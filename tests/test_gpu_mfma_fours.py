"""The matrix-core kernel's staging by fours of cells: widths around four, rows that end in a shifted four, padding that no four
covers, positions in fours (1x1), the forms that keep a cell per lane, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from paper_1608_01409_amd import binding as B
from paper_1608_01409_amd import workloads as wl

pytestmark = pytest.mark.gpu
TOL = 1e-5     # of sum|w*x| per output, as in test_gpu_parity.py


# C, H, W, K, R, S, stride, pad, groups, N
SHAPES = [
    (64, 30, 4, 64, 3, 3, 1, 1, 1, 64), (64, 30, 5, 64, 3, 3, 1, 1, 1, 64), (64, 30, 7, 64, 3, 3, 1, 1, 1, 64),
    (64, 40, 3, 64, 3, 3, 1, 1, 1, 64),                # narrower than four
    (61, 14, 14, 64, 3, 3, 1, 1, 1, 64),               # channels that do not fill an octet
    (130, 9, 9, 70, 5, 5, 1, 2, 2, 40), (96, 27, 27, 64, 3, 3, 2, 1, 1, 24), (96, 28, 28, 64, 3, 3, 2, 0, 1, 24),
    (192, 28, 28, 64, 1, 1, 1, 0, 1, 16), (192, 27, 27, 64, 1, 1, 1, 0, 1, 16), (64, 15, 13, 64, 2, 3, 1, 1, 1, 64),
]


@pytest.mark.parametrize("shape", SHAPES)
def test_layers_against_the_oracle(oracle, shape):
    *dims, N = shape
    layer = wl.small_layer("fours", **dict(zip(("C", "H", "W", "K", "R", "S", "stride", "pad", "groups"), dims)))
    rng = np.random.default_rng(3)
    x = rng.standard_normal((N, layer.C, layer.H, layer.W)).astype(np.float32)
    w = (rng.standard_normal((layer.K, layer.Cg, layer.R, layer.S)) * 0.01).astype(np.float32)
    w[rng.random(w.shape) >= 0.7] = 0
    h = B.sconv_create_csr(layer, w)
    route = B.sconv_route_of(h, N)
    assert route["kernel"] == "mfma", route
    print(f"[gpu-case] {shape} {route}", flush=True)
    out = torch.full((N, layer.K, layer.OH, layer.OW), float("nan"), device="cuda")
    got = B.sconv_forward(h, torch.from_numpy(x).cuda(), out).cpu().numpy()
    ref, ab, _ = oracle.sparse_conv(layer, w, x)
    assert np.all(np.abs(got - ref) <= TOL * ab)
