"""The flat streams on the matrix cores: convolutions against the fp64 oracle, and their errors against the other kernels'."""
import numpy as np
import pytest
import torch

from paper_1608_01409_amd import binding as B
from paper_1608_01409_amd import workloads as wl

pytestmark = pytest.mark.gpu
TOL = 1e-5     # of sum|w*x| per output, as in test_gpu_parity.py


def make(layer, N, density, seed=1, signed=False):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((N, layer.C, layer.H, layer.W)).astype(np.float32)
    if not signed:
        x = np.maximum(x, 0)
    w = (rng.standard_normal((layer.K, layer.Cg, layer.R, layer.S)) * 0.01).astype(np.float32)
    w[rng.random(w.shape) >= density] = 0
    return x, w


def on_matrix_cores(route):
    return route["kernel"] == "flat_mc"


def check(oracle, layer, N, x, w, bias=None, relu=False):
    h = B.sconv_create_csr(layer, w)
    route = B.sconv_route_of(h, N)
    assert on_matrix_cores(route), route
    print(f"[gpu-case] {layer.name} C{layer.C} {layer.H}x{layer.W} K{layer.K} N={N} {route}", flush=True)
    out = torch.full((N, layer.K, layer.OH, layer.OW), float("nan"), device="cuda")
    xd = torch.from_numpy(x).cuda()
    if bias is None:
        B.sconv_forward(h, xd, out)
    else:
        B.sconv_forward_fused(h, xd, torch.from_numpy(bias).cuda(), relu, out)
    got = out.cpu().numpy()
    ref, ab, _ = oracle.sparse_conv(layer, w, x)
    if bias is not None:
        ref, ab = oracle.bias_relu(ref, ab, bias, relu)
    err = np.abs(got.astype(np.float64) - ref)
    bad = ~(err <= TOL * ab + 2.0 ** -149)     # (2^-149: the spacing of the smallest results)
    assert not bad.any(), (route, int(bad.sum()), float(np.nanmax(err / np.maximum(ab, 1e-300))), np.argwhere(bad)[:4])
    return got, ref, route


FIELDS = ("C", "H", "W", "K", "R", "S", "stride", "pad", "groups")


def layer_of(dims):
    return wl.small_layer("mc", **dict(zip(FIELDS, dims)))


# C, H, W, K, R, S, stride, pad, groups, N, density
SHAPES = [
    (256, 13, 13, 384, 3, 3, 1, 1, 1, 70, 0.13),    # several blocks, filters and positions of whole and part workgroups
    (96, 27, 27, 256, 5, 5, 1, 2, 2, 41, 0.13),
    (384, 13, 13, 384, 3, 3, 1, 1, 2, 70, 0.15),
    (192, 28, 28, 128, 3, 3, 1, 1, 1, 33, 0.12),
    (3, 99, 99, 96, 11, 11, 4, 0, 1, 100, 0.30),    # phases of a strided layer, a cell per lane
    (160, 27, 27, 80, 3, 3, 2, 1, 1, 160, 0.10),    # stride on the cells, odd width
    (96, 28, 28, 80, 3, 3, 2, 1, 1, 64, 0.13),      # (0.10 leaves a row of 66 nonzeros)
    (99, 30, 30, 40, 3, 3, 1, 1, 1, 64, 0.20),      # channels that do not fill an octet, 40 filters
    (60, 20, 20, 250, 3, 3, 1, 1, 1, 32, 0.20),
    (99, 20, 20, 150, 3, 3, 1, 1, 1, 32, 0.13),
    (130, 21, 5, 96, 3, 3, 1, 1, 1, 256, 0.19),     # a row of five, the last four of it shifted back
    (300, 7, 7, 150, 3, 3, 1, 1, 1, 256, 0.13),
    (64, 18, 18, 96, 3, 3, 1, 3, 1, 64, 0.20),      # padding as wide as the filter
    (400, 28, 28, 64, 1, 1, 1, 0, 1, 100, 0.30),    # 1x1: positions in fours
    (500, 27, 27, 128, 1, 1, 1, 0, 1, 64, 0.22),    # 1x1: images that no four divides
    (128, 28, 28, 128, 3, 3, 1, 1, 1, 64, 0.20),    # 64 positions a wave
    (192, 14, 14, 96, 3, 3, 1, 1, 1, 256, 0.16),
    (384, 13, 13, 384, 3, 3, 1, 1, 2, 64, 0.50),    # in place of the three-part kernel
    (180, 20, 20, 90, 3, 3, 1, 1, 1, 64, 0.60),
    (472, 12, 12, 356, 3, 3, 1, 1, 1, 34, 0.94),    # channels split over workgroups
]


@pytest.mark.parametrize("shape", SHAPES)
def test_layers_against_the_oracle(oracle, shape):
    *dims, N, density = shape
    layer = layer_of(dims)
    x, w = make(layer, N, density)
    bias = (np.random.default_rng(5).standard_normal(layer.K) * 0.05).astype(np.float32)
    w[1] = 0                                        # an empty row
    check(oracle, layer, N, x, w)
    check(oracle, layer, N, x, w, bias, True)
    check(oracle, layer, N, x, w, bias, False)


# ... and the input channels of a group that pruning took from every filter; -1: the last filter has 18 channels only
PRUNED = [
    (256, 13, 13, 384, 3, 3, 1, 1, 1, 256, 0.20, 0, 96),      # the first channel block without weights
    (256, 13, 13, 384, 3, 3, 1, 1, 1, 70, 0.20, 88, 176),     # one in the middle
    (256, 13, 13, 384, 3, 3, 1, 1, 1, 70, 0.20, 160, 256),    # the last one
    (384, 13, 13, 384, 3, 3, 1, 1, 2, 70, 0.30, 60, 130),
    (400, 28, 28, 64, 1, 1, 1, 0, 1, 100, 0.50, 96, 200),
    (160, 27, 27, 80, 3, 3, 2, 1, 1, 160, 0.15, 30, 90),      # staged a cell per lane
    (472, 12, 12, 356, 3, 3, 1, 1, 1, 34, 0.94, 0, 100),      # channels split over workgroups
    (472, 12, 12, 356, 3, 3, 1, 1, 1, 34, 0.94, 300, 400),
    (256, 13, 13, 385, 3, 3, 1, 1, 1, 70, 0.17, -1, 0),
]


@pytest.mark.parametrize("shape", PRUNED)
def test_channels_without_weights(oracle, shape):
    *dims, N, density, lo, hi = shape
    layer = layer_of(dims)
    x, w = make(layer, N, density)
    if lo < 0:
        w[-1] = 0
        w[-1, :18] = 0.01
    else:
        w[:, lo:hi] = 0
    check(oracle, layer, N, x, w)


MIXED = [(150, 17, 17, 256, 3, 3, 1, 1, 1, 100, 0.18), (99, 20, 20, 150, 3, 3, 1, 1, 1, 32, 0.13), (256, 13, 13, 384, 3, 3, 1, 1, 1, 70, 0.13), (472, 12, 12, 356, 3, 3, 1, 1, 1, 34, 0.94)]


@pytest.mark.parametrize("shape", MIXED)
@pytest.mark.parametrize("what", ["tiny", "huge", "images", "one", "spread", "late", "growing", "zero", "denormal"])
def test_activations_of_every_magnitude(oracle, shape, what):
    """Every output within the tolerance of its own sum of magnitudes, whatever else is in the batch."""
    *dims, N, density = shape
    layer = layer_of(dims)
    x, w = make(layer, N, density)
    rng = np.random.default_rng(7)
    if what == "tiny":
        x *= np.float32(1e-33)
    elif what == "huge":
        x *= np.float32(1e30)
    elif what == "images":                          # image by image 1e-30 ... 1e+30
        x *= (10.0 ** np.linspace(-30, 30, N)).astype(np.float32)[:, None, None, None]
    elif what == "one":                             # one value far above the others, and one below
        x[N // 2, 3, 5, 5] = 1e25
        x[0, 0, 0, 0] = 1e-25
    elif what == "spread":
        x *= (10.0 ** rng.uniform(-20, 20, x.shape)).astype(np.float32)
    elif what == "growing":                         # every few channels sixteen times larger: the scale shrinks with every block
        x *= np.float32(16) ** (np.arange(layer.C) * 20 // layer.C)[None, :, None, None].astype(np.float32)
    elif what == "late":                            # nothing in the channels that the scale is taken from
        x[:, :layer.C - 4] = 0
        x[:, layer.C - 2:] *= np.float32(1e15)
    elif what == "zero":
        x[:] = 0
    else:
        x *= np.float32(1e-39)
    check(oracle, layer, N, x, w)


@pytest.mark.parametrize("shape", MIXED)
@pytest.mark.parametrize("binades", [12, 20, 24, 26, 27, 28, 29, 30, 33])
@pytest.mark.parametrize("alike", [False, True])
def test_small_images_lose_no_bits_beside_large_ones(shape, binades, alike):
    """Image by image as close to 64 bits as the direct kernel's chains where every other image is 2^binades smaller, its
    activations all of about one size: a workgroup's scale leaves them fewer bits, and their sums are taken again.  alike: the
    weights have one sign, so that what is lost adds up."""
    *dims, N, density = shape
    layer = layer_of(dims)
    x, w = make(layer, N, density)
    if alike:
        w = np.abs(w)
    x = np.where(alike | (x > 0), 0.5 + 0.5 * np.random.default_rng(3).random(x.shape), 0).astype(np.float32)
    x[1::2] *= np.float32(2.0 ** -binades)
    xd = torch.from_numpy(x).cuda()
    h = B.sconv_create_csr(layer, w)
    assert on_matrix_cores(B.sconv_route_of(h, N))
    print(f"[gpu-case] small images {layer.name} C{layer.C} K{layer.K} N={N} 2^-{binades}", flush=True)
    exact = torch.nn.functional.conv2d(xd.cpu().double(), torch.from_numpy(w).double(), padding=layer.pad)
    err, chain = ((B.sconv_forward(g, xd).cpu().double() - exact).flatten(1).norm(dim=1) / exact.flatten(1).norm(dim=1)
                  for g in (h, B.sconv_create_csr(layer, w, dict(kernel=2))))
    print(f"[gpu-case] largest ratio {float((err / chain).max()):.3f}", flush=True)
    assert bool((err <= chain).all()), (err / chain).tolist()


# the shortest rows that go there, by what their layer would run on otherwise: C, H = W, stride, K, groups, N, nonzeros, the kernel
# left
SHORTEST = [
    (40, 13, 1, 256, 1, 256, 72, "lds"), (256, 13, 1, 384, 1, 256, 160, "lds"), (384, 13, 1, 384, 2, 96, 740, "mfma"),
    (408, 53, 2, 128, 1, 34, 330, "lds"), (197, 51, 2, 384, 1, 20, 800, "mfma"),     # channel blocks of few steps
]


@pytest.mark.parametrize("case", SHORTEST)
def test_no_row_is_further_off_than_on_the_kernel_that_it_leaves(case):
    """Rows of the least length and others: by length, no further from 64 bits than on the flat-stream kernel with the tiling ranked
    first, or than on the three-part kernel, which serves the same layer with one of its rows shortened."""
    C, hw, stride, K, groups, N, least, left = case
    layer = layer_of((C, hw, hw, K, 3, 3, stride, 1, groups))
    cols = layer.Cg * 9
    rng = np.random.default_rng(21)
    lengths = np.array([least, least + least // 8, 2 * least])[np.arange(K) % 3]
    w = np.zeros((K, cols), np.float32)
    for k in range(K):
        w[k, rng.permutation(cols)[:lengths[k]]] = rng.standard_normal(lengths[k]) * 0.01
    w = w.reshape(K, layer.Cg, 3, 3)
    xd = torch.from_numpy(np.maximum(rng.standard_normal((N, C, hw, hw)), 0).astype(np.float32)).cuda()
    h = B.sconv_create_csr(layer, w)
    route = B.sconv_route_of(h, N)
    assert on_matrix_cores(route), route
    print(f"[gpu-case] shortest rows {case} {route}", flush=True)
    v = w.copy()
    if left == "mfma":
        v[0].reshape(-1)[np.flatnonzero(v[0].reshape(-1))[300:]] = 0
    other = B.sconv_create_csr(layer, v, None if left == "mfma" else B.sconv_rank_plans(h, N, 1)[0])
    if left == "mfma":
        assert B.sconv_route_of(other, N)["kernel"] == "mfma"
    x64, kg = xd.double(), K // groups
    exact = torch.cat([torch.cat([torch.from_numpy(w[g * kg:(g + 1) * kg]).cuda().double().reshape(kg, -1) @ torch.nn.functional.unfold(
        x64[i:i + 1, g * layer.Cg:(g + 1) * layer.Cg], (3, 3), padding=1, stride=stride)[0] for g in range(groups)])[None] for i in range(N)])
    err, was = (((B.sconv_forward(g, xd).double().flatten(2) - exact).transpose(0, 1).flatten(1).norm(dim=1) /
                 exact.transpose(0, 1).flatten(1).norm(dim=1)).cpu().numpy() for g in (h, other))
    for n in np.unique(lengths):
        rows = np.flatnonzero((lengths == n) & (np.arange(K) > 0))
        ratio = err[rows] / was[rows]
        print(f"[gpu-case] {n} nonzeros: {err[rows].mean():.3g} / {was[rows].mean():.3g}, ratio {ratio.mean():.3f}", flush=True)
        # (the ratio scatters by 0.07-0.1 from row to row)
        assert ratio.mean() <= 1 + 3 * 0.1 / np.sqrt(len(rows)), (n, ratio.mean())
        if n > least:
            assert ratio.mean() <= 1, (n, ratio.mean())


@pytest.mark.parametrize("shape", MIXED)
def test_infinities_meet_stored_weights_only(shape):
    """Infinities, NaN and values near the largest: the outputs the direct kernel gives, stored zeros included."""
    *dims, N, density = shape
    layer = layer_of(dims)
    x, w = make(layer, N, density, signed=True)
    rng = np.random.default_rng(9)
    for v in (np.inf, -np.inf, np.nan, 3e38, -3e38):
        for _ in range(3):
            x[rng.integers(N), rng.integers(layer.C), rng.integers(layer.H), rng.integers(layer.W)] = v
    cols = layer.Cg * layer.R * layer.S
    rowptr, colidx, values = [0], [], []
    for k in range(layer.K):
        (j,) = np.nonzero(w.reshape(layer.K, cols)[k])
        v = w.reshape(layer.K, cols)[k][j].copy()
        v[::50] = 0
        colidx.extend(j), values.extend(v), rowptr.append(len(colidx))
    bias = torch.from_numpy((rng.standard_normal(layer.K) * 0.05).astype(np.float32)).cuda()
    xd = torch.from_numpy(x).cuda()
    h = B.sconv_create_csr_from_arrays(layer, rowptr, colidx, values)
    direct = B.sconv_create_csr_from_arrays(layer, rowptr, colidx, values, dict(kernel=2))
    assert on_matrix_cores(B.sconv_route_of(h, N))
    for b, relu in ((None, False), (bias, False), (bias, True)):
        got = B.sconv_forward_fused(h, xd, b, relu).cpu().numpy()
        want = B.sconv_forward_fused(direct, xd, b, relu).cpu().numpy()
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
        assert np.array_equal(np.sign(got[np.isinf(got)]), np.sign(want[np.isinf(want)]))
        finite = np.isfinite(want)
        largest = np.where(np.isfinite(x), np.abs(x), 0).max(axis=(1, 2, 3)).astype(np.float64)   # of an image
        scale = np.abs(w).reshape(layer.K, -1).sum(1)[None, :, None, None] * largest[:, None, None, None]
        assert np.all(np.abs(got[finite].astype(np.float64) - want[finite]) <= (np.broadcast_to(scale, want.shape)[finite] + 1) * TOL)


def test_without_allocation_and_under_capture():
    """sconv_forward_noalloc gives sconv_forward's bits, also replayed from a graph between other calls."""
    *dims, N, density = MIXED[0]
    layer = layer_of(dims)
    x, w = make(layer, N, density)
    h = B.sconv_create_csr(layer, w)
    assert on_matrix_cores(B.sconv_route_of(h, N))
    xd = torch.from_numpy(x).cuda()
    want = B.sconv_forward(h, xd)
    out = torch.full_like(want, float("nan"))
    B.sconv_forward_noalloc(h, xd, out)
    assert torch.equal(out, want)
    s = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        B.sconv_forward_noalloc(h, xd, out, stream=torch.cuda.current_stream())
    for i in range(3):
        xd.mul_(1.0 + i)
        want = B.sconv_forward(h, xd)
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), i


def test_short_rows_and_unfit_weights_stay_on_the_vector_units():
    """Layers with rows of fewer than 16 nonzeros, or weights that lie too far apart, keep the chains."""
    *dims, N, density = MIXED[0]
    layer = layer_of(dims)
    _, w = make(layer, 1, density)
    assert on_matrix_cores(B.sconv_route_of(B.sconv_create_csr(layer, w), N))
    for change in ("short", "small", "inf"):
        v = w.copy()
        if change == "short":
            v[3] = 0
            v[3, :15, 0, 0] = 1
        else:
            v[3, 0, 0, 0] = 1e-12 if change == "small" else np.inf
        assert B.sconv_route_of(B.sconv_create_csr(layer, v), N)["kernel"] in ("flat", "flow"), change
