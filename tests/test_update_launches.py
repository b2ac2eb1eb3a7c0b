"""The update's launches, with the HIP runtime replaced on the CPU (tests/host/update_launches.cpp)."""
import os
import subprocess

import pytest

from paper_2608_24067_amd import build as hipbuild

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(not os.path.exists(hipbuild.HIPCC), reason="needs hipcc")
def test_lds_limits_are_the_same_for_every_update(tmp_path):
    def run(*cmd):
        r = subprocess.run(cmd, cwd=ROOT, capture_output=True, text=True, timeout=600)
        assert r.returncode == 0, f"{' '.join(cmd)}\n{r.stdout}\n{r.stderr}"
        return r

    device, main = str(tmp_path / "som_update.o"), str(tmp_path / "main.o")
    run(hipbuild.HIPCC, f"--offload-arch={hipbuild.ARCH}", "--offload-host-only", "-fuse-cuid=none", "-O1", "-fPIC",
        "-std=c++17", "-Iinclude", "-c", "paper_2608_24067_amd/csrc/som_update.hip", "-o", device)
    run("g++", "-std=c++17", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-Iinclude", "-fPIC", "-c",
        "tests/host/update_launches.cpp", "-o", main)
    exe = str(tmp_path / "update_launches")
    run("g++", device, main, "-o", exe)
    assert "passed" in run(exe).stdout
