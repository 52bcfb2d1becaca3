"""Host rules for grids of blocks (m1_grid.h), compiled by the host compiler and called on the CPU."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1806_07390_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("grid")
    src = d / "grid.cpp"
    src.write_text('#include "m1_grid.h"\n'
                   'extern "C" long stride_blocks(long need, long step, long entries, int per_cu, int cus) {\n'
                   '  return (long)fm1::stride_blocks(need, step, entries, per_cu, cus);\n}\n')
    so = str(d / "grid.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", so])
    lib = ctypes.CDLL(so)
    lib.stride_blocks.argtypes = [ctypes.c_long] * 3 + [ctypes.c_int] * 2
    lib.stride_blocks.restype = ctypes.c_long
    return lib


# zones x groups, the step tiling's blocks, blocks that hold every zone once
@pytest.mark.parametrize("step_blocks,need", [(728, 14746), (494, 6554), (10, 40000), (3528, 100000)])
@pytest.mark.parametrize("per_cu", [4, 6])
def test_stride_blocks_fill_the_chip(lib, step_blocks, need, per_cu):
    nb = lib.stride_blocks(need, step_blocks, need, per_cu, 256)
    assert nb >= 256 * per_cu and nb >= step_blocks and nb <= need


def test_stride_blocks_bounds(lib):
    assert lib.stride_blocks(3, 1, 3, 4, 256) == 3            # a small grid: every zone once
    assert lib.stride_blocks(9000, 100, 300, 4, 256) == 300   # never past the scratch
    assert lib.stride_blocks(0, 0, 0, 4, 256) == 1
    assert lib.stride_blocks(9000, 100, 9000, 4, 0) == 1024   # unknown device
