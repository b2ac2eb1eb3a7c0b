"""The rules that choose a path or a launch by sizes, built for the host (tests/host/rules.cpp)."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RESIDENT = 1024  # sweep workgroups the chip holds: 256 compute units, four each

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                                reason="needs g++ and the ROCm headers")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("rules") / "librules.so")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-Iinclude", "tests/host/rules.cpp", "-o", out], cwd=ROOT, check=True)
    lib = ctypes.CDLL(out)
    i64, i32 = ctypes.c_int64, ctypes.c_int32
    lib.group_tiles.argtypes, lib.group_tiles.restype = [i64, i64, i32, i32], i64
    lib.strips.argtypes, lib.strips.restype = [i64, i32], i64
    return lib


@pytest.mark.parametrize("f16", [0, 1])
def test_long_tile_groups_leave_enough_workgroups(rules, f16):
    """Groups above four tiles only where the launch still has many rounds of resident workgroups: a map of one
    strip and 1,500 tiles would otherwise leave compute units idle, one of 6,000 tiles half of them."""
    for M in (1, 256, 512, 513, 1024, 4096, 16384, 65025, 1 << 20):
        strips = rules.strips(M, 8)
        for nt in (1, 2, 187, 1499, 1500, 3000, 5999, 6000, 12000, 12500, 19999, 20000, 30000, 31250, 62500, 125000,
                   250000, 1 << 28):
            g = rules.group_tiles(nt, strips, 8, f16)
            assert g % 4 == 0 and 4 <= g <= 32
            assert g == 4 or -(-nt // g) * strips >= 8 * RESIDENT, (M, nt, g)


def test_tile_groups_of_many_strips_are_long(rules):
    assert rules.group_tiles(62500, 2048, 8, 0) == 8 and rules.group_tiles(62500, 2048, 8, 1) == 32
    assert rules.group_tiles(2000, 2048, 8, 1) == 8 and rules.group_tiles(31250, 8, 8, 0) == 8
