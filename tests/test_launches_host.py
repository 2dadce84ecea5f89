"""Host logic of the C-ABI library with stand-ins for the HIP runtime and the
kernels (tests/host/check_launches.cpp): the launches of contexts on several
streams.  No GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1902_11193_amd", "csrc")
CXX = "/opt/rocm/bin/amdclang++"


def test_launches_of_several_contexts(tmp_path):
    if not os.path.exists(CXX):
        pytest.skip("amdclang++ not available")
    exe = tmp_path / "check_launches"
    subprocess.run([CXX, "-O1", "-std=c++17", "-Wno-unused-value", "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I",
                    os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "host", "check_launches.cpp"),
                    os.path.join(CSRC, "lbm_capi.cpp"), os.path.join(CSRC, "lbm_host.cpp"), "-o", str(exe),
                    "-lpthread"], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "bad 0" in r.stdout
