"""Host check of the flat streams packed for the matrix cores (tests/host/flat_mc_check.cpp).  No GPU."""
import os
import shutil
import subprocess

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
