"""A 1D plan begun while its stream is captured, on the CPU (tests/host/capture1d.cpp)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2505_10857_amd")


def test_begin_under_capture_is_refused_and_leaves_the_plan_usable(tmp_path):
    """Beginning a plan uploads its tables from host memory that the plan owns, so it cannot be
    recorded; and a refused begin must not count as an upload for the next one."""
    lib = os.path.join(PKG, "libnmg.so")
    if not os.path.exists(lib):
        pytest.skip("libnmg.so not built (run __graft_entry__.build())")
    exe = str(tmp_path / "capture1d")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "host", "capture1d.cpp"),
                           lib, "-Wl,-rpath," + PKG, "-Wl,-rpath-link,/opt/rocm/lib", "-o", exe])
    out = subprocess.run([exe], text=True, capture_output=True, check=True).stdout.split()
    captured, recorded, after, copied, fresh, fresh_copied = map(int, out)
    from paper_2505_10857_amd import _abi as A
    assert captured == A.NMG_EHIP and recorded == 0
    assert after == fresh == A.NMG_OK
    assert copied == fresh_copied > 1000
