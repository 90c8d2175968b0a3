"""Unpadded layers whose stride is a multiple of four on the flat streams of the matrix cores: four columns of the input a load, single
ones where four could pass the input's end, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from paper_1608_01409_amd import binding as B

from .test_gpu_flat_mc import check, layer_of, make

pytestmark = pytest.mark.gpu

# C, H, W, K, R, S, stride, pad, groups, N, density
SHAPES = [
    (3, 99, 99, 96, 11, 11, 4, 0, 1, 100, 0.30),     # the last cell's fours pass the end of a row, and of the input
    (3, 99, 100, 96, 11, 11, 4, 0, 1, 100, 0.30),    # rows of whole fours
    (3, 97, 101, 96, 11, 11, 4, 0, 1, 100, 0.30),
    (10, 46, 77, 75, 10, 10, 4, 0, 1, 150, 0.47),
    (24, 39, 73, 166, 12, 7, 4, 0, 2, 64, 0.45),     # groups; a last tap that not every column has
    (11, 49, 50, 69, 9, 13, 4, 0, 1, 150, 0.33),     # channels split over workgroups
    (12, 75, 101, 144, 12, 4, 4, 0, 1, 150, 0.23),   # one tap along a row
    (11, 25, 97, 87, 6, 9, 4, 0, 1, 150, 0.48),      # few rows
    (12, 97, 109, 270, 12, 13, 8, 0, 2, 150, 0.36),  # eight columns a row of the phases
    (39, 53, 30, 196, 3, 10, 4, 0, 1, 61, 0.37),     # fewer filter rows than the stride: fours of phases that no weight has
    (34, 32, 83, 273, 2, 8, 4, 0, 1, 115, 0.588),
    (34, 22, 94, 285, 7, 18, 8, 0, 1, 71, 0.139),
]


@pytest.mark.parametrize("shape", SHAPES)
def test_against_the_oracle(oracle, shape):
    *dims, N, density = shape
    layer = layer_of(dims)
    x, w = make(layer, N, density, signed=True)
    check(oracle, layer, N, x, w)


def test_values_that_no_tap_reads(oracle):
    """Rows and columns behind the last tap, and what lies behind the input in memory, are loaded and meet no stored weight."""
    layer = layer_of((3, 102, 102, 96, 11, 11, 4, 0, 1))
    N = 100
    x, w = make(layer, N, 0.3, signed=True)
    used = 4 * (layer.OH - 1) + 11
    x[:, :, used:] = np.inf
    x[:, :, :, used:] = np.nan
    h = B.sconv_create_csr(layer, w)
    assert B.sconv_route_of(h, N)["kernel"] == "flat_mc"
    room = torch.full((x.size + 64,), float("inf"), device="cuda")
    room[:x.size] = torch.from_numpy(x.reshape(-1))
    out = torch.full((N, layer.K, layer.OH, layer.OW), float("nan"), device="cuda")
    B.sconv_forward(h, room[:x.size].view(x.shape), out)
    clean = np.where(np.isfinite(x), x, np.float32(0))
    ref, ab, _ = oracle.sparse_conv(layer, w, clean)
    err = np.abs(out.cpu().numpy().astype(np.float64) - ref)
    assert (err <= 1e-5 * ab + 2.0 ** -149).all()
