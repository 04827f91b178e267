"""What a plan's calls launch and how much scratch they hold, on the CPU: the directed cases of
tests/sanitize/host_san.cpp (the library's host code under ASan / UBSan, stand-in HIP calls, launchers
that touch the scratch as the kernels do)."""
import os
import shutil
import subprocess

import pytest

from test_host_sanitizers import ROOT, SAN, run

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("routes") / "host_san")
    csrc = os.path.join(ROOT, "paper_2311_03285_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", *SAN, "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I" + os.path.join(ROOT, "include"), "-I" + csrc, os.path.join(ROOT, "tests", "sanitize", "host_san.cpp"),
                           os.path.join(csrc, "pool.cpp"), os.path.join(csrc, "plan.cpp"), "-o", out])
    return out


@pytest.mark.parametrize("case", ["failed_apply", "static_route", "scratch_is_sized_once", "fuse_decode_never",
                                  "y_in_the_buffer_of_x", "expand_runs", "slots_of_the_call", "larger_items",
                                  "larger_items_pay", "larger_items_in_fours", "larger_items_of_no_call", "expand_lds", "shrink_pages_of_the_caller", "hand_over", "hand_over_pays",
                                  "words_of_the_calls_that_use_them"])
def test_case(exe, case):
    assert f"host_san OK: {case}" in run(exe, case)
