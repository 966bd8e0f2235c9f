"""Which plans run two chains of launches (CPU only): the launches of a step
of ``csrc/abi.cpp``, linked with host-only stand-ins for the HIP runtime and
the kernel launchers, on both sides of every line of the rule; and every
launch failing in turn, with nothing left unjoined on the second stream.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_plan_chains(tmp_path):
    gxx = shutil.which("g++")
    if not gxx or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"):
        pytest.skip("g++ or the HIP headers are not available")
    exe = str(tmp_path / "chains_driver")
    subprocess.check_call([gxx, "-std=c++17", "-g", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-o", exe,
                           os.path.join(HERE, "sanitize", "chains_driver.cpp"),
                           os.path.join(ROOT, "paper_2508_06768_amd", "csrc", "abi.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "chains driver: ok" in r.stdout
