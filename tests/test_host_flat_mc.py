"""Host check of the flat streams packed for the matrix cores (tests/host/flat_mc_check.cpp).  No GPU."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_1608_01409_amd import binding as B
from paper_1608_01409_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1608_01409_amd")


def test_records_as_the_kernel_reads_them(tmp_path):
    """Random layers in every form the kernel takes (strides, phases, groups, empty and dense rows, stored zeros): each weight
    once, in a place the matrix instruction allows, and every LDS address inside the staged block."""
    cxx = shutil.which("g++")
    assert cxx, "needs the host compiler"
    exe = tmp_path / "flat_mc_check"
    subprocess.check_call([cxx, "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                           os.path.join(ROOT, "tests", "host", "flat_mc_check.cpp"), "-L", PKG, "-l:libsconv.so", f"-Wl,-rpath,{PKG}",
                           "-Wl,-rpath-link,/opt/rocm/lib", "-o", str(exe)])
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-4000:] + res.stderr[-2000:]


# channels, height and width, batch, density, filters of a group, groups; what they took on the three-part kernel and here, us
@pytest.mark.parametrize("c,hw,n,density,per_group,groups,there", [
    (114, 54, 87, 0.72, 15, 2, False),   # 225 266
    (131, 41, 89, 0.65, 24, 1, False),   # 165 190
    (278, 53, 25, 0.74, 18, 2, False),   # 163 204
    (164, 26, 108, 0.88, 12, 1, False),  # 99 126
    (204, 15, 88, 0.48, 17, 2, False),   # 47 58
    (246, 23, 45, 0.45, 97, 2, True),    # 179 147
    (472, 21, 106, 0.454, 39, 2, True),  # 300 195
])
def test_few_filters_stay_on_the_three_part_kernel(c, hw, n, density, per_group, groups, there):
    """Filters that fill two row tiles at most keep a wave waiting for columns: slower than the three-part kernel."""
    layer = wl.Layer("few", C=c, H=hw, W=hw, K=groups * per_group, R=5, S=5, stride=1, pad=2, groups=groups)
    rng = np.random.default_rng(3)
    w = rng.standard_normal((layer.K, layer.Cg, 5, 5), dtype=np.float32)
    w[rng.random(w.shape) >= density] = 0
    route = B.sconv_route_of(B.sconv_create_csr(layer, w), n)
    assert route["kernel"] == ("flat_mc" if there else "mfma"), route


def test_the_shortest_row_decides():
    """A layer whose rows are long on average and whose shortest one is not keeps the sums that are good enough for that one."""
    def route(c, groups, n, density, length):
        layer = wl.Layer("rows", C=c, H=13, W=13, K=384, R=3, S=3, stride=1, pad=1, groups=groups)
        rng = np.random.default_rng(5)
        w = rng.standard_normal((layer.K, layer.Cg, 3, 3), dtype=np.float32)
        w[rng.random(w.shape) >= density] = 0
        if length:
            w[7].reshape(-1)[np.flatnonzero(w[7])[length:]] = 0
        if length == 0:
            w[7] = 0
        return B.sconv_route_of(B.sconv_create_csr(layer, w), n)

    full = route(256, 1, 256, 0.12, None)
    assert full["kernel"] == "flat_mc" and full["nt"] == 4, full
    for length, nt in ((0, 4), (160, 4), (159, 2), (72, 2), (71, 1), (16, 1)):
        r = route(256, 1, 256, 0.12, length)
        assert r["kernel"] in (("flat_mc",) if nt > 1 else ("flat", "flow")) and r["nt"] == nt, (length, r)
    for length, there in ((None, True), (0, True), (740, True), (739, False), (100, False)):
        r = route(384, 2, 256, 0.5, length)
        assert r["kernel"] == ("flat_mc" if there else "mfma"), (length, r)
