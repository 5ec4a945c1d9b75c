"""The library's host code over a stand-in for the HIP runtime
(host_runtime.h): what one GPU or a healthy runtime cannot show."""
import os
import shutil
import subprocess

import pytest

from paper_2408_15654_amd import lbm

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TESTS = os.path.join(ROOT, "tests")


@pytest.fixture(scope="module")
def host_check(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    lbm.load()
    exe = tmp_path_factory.mktemp("host") / "host_check"
    lib = os.path.join(ROOT, "paper_2408_15654_amd", "liblbm.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-rdynamic", "-pthread", "-I", TESTS, "-I",
                           os.path.join(ROOT, "include"), os.path.join(TESTS, "host_check.cpp"),
                           lib, "-Wl,-rpath," + os.path.dirname(lib),
                           "-Wl,--allow-shlib-undefined", "-o", str(exe)])
    return str(exe)


@pytest.mark.parametrize("check", ["other_device", "other_device_batch", "failed_chunk", "side_by_side",
                                   "no_more_streams", "launch_parity", "one_step_launches", "two_rounds", "two_step_tiles",
                                   "tile_plan",
                                   "unaligned_fields", "pinned_memory", "first_transfers",
                                   "staged_writes", "batch_transfers"])
def test_host_code(host_check, check):
    out = subprocess.run([host_check, check], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and check + " ok" in out.stdout, (out.returncode, out.stdout,
                                                                 out.stderr)


def test_step_plan_of_no_handle():
    import ctypes

    steps = ctypes.c_int32(7)
    assert lbm.load().lbm_step_plan(None, ctypes.byref(steps)) == b"lbm_step_kernel"
    assert steps.value == 7
    assert lbm.load().lbm_step_plan(None, None) == b"lbm_step_kernel"
