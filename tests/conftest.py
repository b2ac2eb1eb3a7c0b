import ctypes
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")
    config.addinivalue_line("markers", "slow: long-running (full-size workloads)")


def gpu_available() -> bool:
    try:
        import torch
        return torch.cuda.is_available()
    except Exception:
        return False


@pytest.fixture(scope="session")
def rules(tmp_path_factory):
    """The rules that choose a path or a launch by sizes, built for the host (tests/host/rules.cpp)."""
    out = str(tmp_path_factory.mktemp("rules") / "librules.so")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-Iinclude", "tests/host/rules.cpp", "-o", out], cwd=ROOT, check=True)
    lib = ctypes.CDLL(out)
    i64, i32 = ctypes.c_int64, ctypes.c_int32
    lib.group_tiles.argtypes, lib.group_tiles.restype = [i64, i64, i32, i32], i64
    lib.rows_direct.argtypes = [i64, i64, i64, i32, i32]
    lib.regroups.argtypes = [i64, i64, i64, i32]
    lib.strips.argtypes, lib.strips.restype = [i64, i32], i64
    return lib


@pytest.fixture(scope="session")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test collected without a visible GPU")
    return torch.device("cuda:0")
