"""Host checks of which kernel a call goes to (tests/host/dispatch_check.cpp): the library's own dispatch with its launches
and uploads replaced, so that nothing needs a GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1608_01409_amd")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    cxx = shutil.which("g++")
    assert cxx, "needs the host compiler"
    exe = tmp_path_factory.mktemp("dispatch") / "dispatch_check"
    subprocess.check_call([cxx, "-O1", "-g", "-std=c++17", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                           os.path.join(ROOT, "tests", "host", "dispatch_check.cpp"), "-L", PKG, "-l:libsconv.so", f"-Wl,-rpath,{PKG}",
                           "-Wl,-rpath-link,/opt/rocm/lib", "-ldl", "-o", str(exe)])
    return str(exe)


def run(program, what):
    res = subprocess.run([program, what], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-4000:] + res.stderr[-2000:]


def test_a_measured_choice_is_kept(program):
    """sconv_tune and sconv_fc_tune hold for their batch size, whatever other batch sizes follow."""
    run(program, "tuned")


def test_the_choice_for_a_batch_size_does_not_depend_on_what_ran_before(program):
    run(program, "untuned")


def test_the_call_without_allocation_takes_what_is_prepared(program):
    """sconv_forward_noalloc after sconv_forward: the same kernels, for batch sizes that share a tiling as well, and for as
    long as the tiling is remembered."""
    run(program, "prepared")


def test_a_kernel_whose_arrays_find_no_room_is_not_taken(program):
    run(program, "no_room")


def test_layers_of_many_short_rows_stay_off_the_matrix_cores(program):
    run(program, "short_rows")


def test_the_first_call_uploads_what_it_reads(program):
    run(program, "first_call")


def test_the_route_is_what_a_call_launches(program):
    run(program, "routes")


def test_calls_that_measured_slower_on_a_gather_kernel_do_not_go_there(program):
    run(program, "gather_limits")


def test_a_tiling_that_no_call_runs_is_not_packed(program):
    run(program, "unpacked_tilings")


def test_the_flat_streams_on_the_matrix_cores(program):
    run(program, "flat_mc")


def test_layers_of_one_tap_keep_their_precision(program):
    """The column kernel takes no call from a kernel whose sums are closer to the exact ones."""
    run(program, "one_tap_limits")


def test_layers_of_one_tap_run_the_column_kernel(program):
    """The route names the matrix cores for both of its kernels: which of them a call launches is seen here."""
    run(program, "column_calls")
