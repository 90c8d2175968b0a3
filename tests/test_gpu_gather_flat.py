"""The four-position gather kernel with its fours counted through the image, and through each row of layers that could have them so: rows
that end anywhere in a four, images that end in one, filters of both orientations, and no more of the neighbouring memory than before."""
import numpy as np
import pytest
import torch

from paper_1608_01409_amd import binding as B
from paper_1608_01409_amd import workloads as wl

pytestmark = pytest.mark.gpu
TOL = 1e-5

# C, H, W, K, R, S, pad, groups, N (S = 2 pad + 1: an output row is as long as an input row)
BY_ROW = [(12, 13, 13, 24, 3, 3, 1, 1, 4), (9, 14, 14, 20, 3, 3, 1, 1, 10), (20, 7, 5, 16, 3, 3, 1, 2, 10), (7, 9, 9, 16, 1, 1, 0, 1, 5),
         (6, 10, 6, 8, 5, 5, 2, 1, 7), (5, 9, 5, 8, 2, 3, 1, 1, 9), (8, 5, 13, 12, 5, 3, 1, 1, 11), (3, 6, 7, 8, 3, 7, 3, 1, 13), (4, 31, 5, 8, 1, 5, 2, 2, 4)]
# with so many filters that the image's fours are a round of 256 workgroups less; each number of waves a row
BY_IMAGE = [(12, 13, 13, 65, 3, 3, 1, 1, 4), (12, 13, 13, 129, 3, 3, 1, 1, 4), (9, 14, 14, 29, 3, 3, 1, 1, 10), (9, 14, 14, 225, 3, 3, 1, 1, 10),
            (20, 7, 5, 86, 3, 3, 1, 2, 10), (7, 9, 9, 341, 1, 1, 0, 1, 5), (6, 10, 6, 86, 5, 5, 2, 1, 7), (5, 9, 5, 86, 2, 3, 1, 1, 9),
            (8, 5, 13, 171, 5, 3, 1, 1, 11), (3, 6, 7, 103, 3, 7, 3, 1, 13), (4, 31, 5, 206, 1, 5, 2, 2, 4), (60, 13, 13, 70, 3, 3, 1, 1, 4)]
CASES = BY_ROW + BY_IMAGE


def workgroups_of_fullest_cu(fours, K, splits):
    return -(-(-(-fours // 64) * -(-K // max(1, 4 // splits))) // 256)


@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_fours_through_the_image(oracle, case):
    C, H, W, K, R, S, pad, groups, N = case
    layer = wl.small_layer("flat", C=C, H=H, W=W, K=K, R=R, S=S, pad=pad, groups=groups)
    by_image, by_row = -(-layer.OH * W // 4), layer.OH * -(-W // 4)
    assert layer.OW == W and -(-N * by_image // 64) < -(-N * by_row // 64)
    rng = np.random.default_rng(C * H + W)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = np.where(rng.random((K, layer.Cg, R, S)) < 0.5, rng.standard_normal((K, layer.Cg, R, S)), 0).astype(np.float32)
    print(f"[gpu-case] gather flat {case}", flush=True)
    h = B.sconv_create_csr(layer, w)
    route = B.sconv_route_of(h, N)
    assert route["kernel"] == "gather4"
    through_image = workgroups_of_fullest_cu(N * by_image, K, route["splits"]) < workgroups_of_fullest_cu(N * by_row, K, route["splits"])
    assert through_image == (case in BY_IMAGE)
    ref, ab, _ = oracle.sparse_conv(layer, w, x)
    around = torch.full((x.size + 2 * 4096,), float("nan"), device="cuda")          # no window may see what lies beside the input
    xd = around[4096:4096 + x.size].view(x.shape)
    xd.copy_(torch.from_numpy(x))
    out = torch.full((N + 2, K, layer.OH, layer.OW), float("nan"), device="cuda")
    got = B.sconv_forward(h, xd, out[1:-1]).cpu().numpy()
    assert np.all(np.abs(got.astype(np.float64) - ref) <= TOL * ab) and np.all(got[ab == 0] == 0)
    assert out[0].isnan().all() and out[-1].isnan().all()
    # an infinity in a corner is seen by the windows over it only
    x[N - 1, C - 2, H - 1, W - 1] = x[0, 1, 0, 0] = np.inf
    xd.copy_(torch.from_numpy(x))
    got = B.sconv_forward(h, xd).cpu()
    want = B.sconv_forward(B.sconv_create_csr(layer, w, dict(kernel=2)), xd).cpu()
    assert torch.equal(got.isinf(), want.isinf()) and torch.equal(got.isnan(), want.isnan())
