"""The split of iso-parametric meshes into launches (host code, built with the host
compiler): meshes whose work-groups would be 2^32 threads or more in one launch, and
plans of up to 64 blocks (tests/iso_launch_driver.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                    reason="needs the host compiler and the HIP headers")
def test_iso_launches(tmp_path):
    exe = str(tmp_path / "iso_launch")
    flags = ["-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include")]
    r = subprocess.run(["g++"] + flags + [os.path.join(ROOT, "tests", "iso_launch_driver.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and "ok: 0 failures" in r.stdout, r.stdout[-4000:]
