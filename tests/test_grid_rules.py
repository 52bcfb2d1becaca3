"""Host rules for grids of blocks (m1_grid.h), compiled by the host compiler and called on the CPU."""
import ctypes
import os
import shutil
import subprocess

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1806_07390_amd", "libfornax_m1.so")
CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1806_07390_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("grid")
    src = d / "grid.cpp"
    src.write_text('#include "m1_grid.h"\n'
                   'extern "C" long stride_blocks(long need, long step, long entries, int per_cu, int cus) {\n'
                   '  return (long)fm1::stride_blocks(need, step, entries, per_cu, cus);\n}\n'
                   'extern "C" int plane_kernel_pays(long c3b, int c3tm, long tb, int tthr, int ttm, int n2, int sph, int mm, int ppm,\n'
                   '                                 int m1s, int cus) {\n'
                   '  return fm1::plane_kernel_pays(c3b, c3tm, tb, tthr, ttm, n2, sph, mm, ppm, m1s, cus);\n}\n')
    so = str(d / "grid.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", so])
    lib = ctypes.CDLL(so)
    lib.stride_blocks.argtypes = [ctypes.c_long] * 3 + [ctypes.c_int] * 2
    lib.stride_blocks.restype = ctypes.c_long
    lib.plane_kernel_pays.argtypes = [ctypes.c_long, ctypes.c_int, ctypes.c_long] + [ctypes.c_int] * 8
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


class C3Tile(ctypes.Structure):
    _fields_ = [(k, ctypes.c_int) for k in ("NR", "TM", "RT", "ntx", "nty", "ntz", "ngb", "nblocks", "xq", "xr")]


def _ceil(a, b):
    return -(-a // b)


def _tiles(n, G, sph):
    """Blocks and planes of the plane kernel (8 rows, 256 CUs) and of the tiled kernel in double."""
    rt = {1: 4, 2: 2}.get(G, 1)
    col = _ceil(_ceil(n[0], 14), rt) * _ceil(n[1], 8) * _ceil(G, 4)
    best = None
    for tm in range(min(8, n[2]), n[2] + 1):
        nb = col * _ceil(n[2], tm)
        cost = _ceil(nb, 256) * (tm + 3)
        if best is None or cost <= best[0]:
            best = (cost, nb, tm)
    gb = 2 if sph else 4
    while G % gb:
        gb -= 1
    tx, ty = (16, 8) if sph else (8, 8)
    nb = _ceil(n[0], tx - 2) * _ceil(n[1], ty - 2) * _ceil(n[2], 16) * (G // gb)
    return best[1], best[2], nb, tx * ty * gb, 16


# (grid, groups, spherical, limiter, M1 speeds, whether the plane kernel measured faster)
MEASURED = [((8, 8, 8), 1, 0, 0, 0, 0), ((8, 8, 8), 3, 0, 0, 0, 0), ((33, 32, 8), 5, 0, 1, 0, 0),
            ((90, 70, 8), 1, 0, 0, 0, 0), ((180, 160, 8), 5, 0, 0, 0, 0), ((12, 12, 12), 3, 0, 0, 0, 1),
            ((24, 24, 24), 1, 0, 1, 0, 1), ((10, 10, 11), 1, 0, 3, 0, 0), ((10, 10, 11), 3, 0, 0, 0, 1),
            ((16, 16, 16), 3, 0, 3, 0, 1), ((90, 70, 60), 10, 0, 0, 0, 1), ((75, 61, 53), 10, 0, 0, 0, 1),
            ((90, 70, 8), 9, 0, 0, 0, 1), ((32, 8, 8), 3, 1, 0, 0, 0), ((128, 48, 10), 3, 1, 0, 0, 0),
            ((48, 12, 16), 9, 1, 0, 0, 1), ((256, 64, 64), 5, 1, 0, 0, 1), ((32, 8, 8), 1, 1, 1, 0, 0),
            ((80, 24, 64), 5, 1, 1, 0, 0), ((256, 64, 64), 5, 1, 1, 0, 0), ((180, 64, 96), 3, 1, 1, 0, 0),
            ((256, 64, 64), 10, 1, 3, 0, 0), ((128, 48, 10), 13, 1, 1, 0, 1), ((96, 32, 48), 9, 1, 1, 0, 1),
            ((96, 32, 48), 9, 1, 3, 0, 1), ((180, 64, 96), 15, 1, 1, 0, 1), ((90, 70, 60), 5, 0, 0, 0, 1),
            ((10, 10, 10), 1, 0, 0, 1, 0), ((12, 12, 12), 3, 0, 0, 1, 1), ((180, 64, 96), 3, 1, 0, 1, 0),
            ((32, 8, 16), 9, 1, 1, 0, 1), ((40, 10, 12), 9, 1, 1, 0, 0), ((48, 12, 16), 9, 1, 0, 1, 1)]


@pytest.mark.parametrize("n,G,sph,lim,ws,fast", MEASURED)
def test_plane_kernel_where_it_measured_faster(lib, n, G, sph, lim, ws, fast):
    c3b, c3tm, tb, tthr, ttm = _tiles(n, G, sph)
    assert bool(lib.plane_kernel_pays(c3b, c3tm, tb, tthr, ttm, n[2], sph, lim == 0, lim == 3, ws, 256)) == bool(fast)


# (grid, groups, spherical, limiter, whether Step 1 of the velocity step measured faster on the plane kernel)
VELOCITY = [((20, 20, 20), 17, 0, 1, 0), ((20, 20, 20), 17, 0, 0, 1), ((30, 28, 28), 6, 0, 1, 0), ((50, 40, 40), 9, 0, 1, 1),
            ((20, 20, 20), 12, 0, 1, 1), ((64, 32, 32), 4, 1, 1, 0), ((64, 32, 32), 4, 1, 0, 1),
            ((128, 48, 64), 1, 1, 1, 0), ((96, 32, 48), 12, 1, 1, 1), ((32, 8, 8), 12, 1, 0, 0)]


@pytest.mark.skipif(not os.path.exists(LIB), reason="library not built (run __graft_entry__.build())")
@pytest.mark.parametrize("n,G,sph,lim,fast", VELOCITY)
def test_velocity_step1_where_it_measured_faster(n, G, sph, lim, fast):
    from paper_1806_07390_amd import m1
    fn = m1._lib._ZN3fm118choose_c3_vel_tileERK14fornax_m1_desci
    fn.argtypes, fn.restype = [ctypes.POINTER(m1.Desc), ctypes.c_int], C3Tile
    d = m1.Desc()
    d.ndim, d.n[:], d.ngroups, d.coord, d.limiter, d.precision, d.c = 3, list(n), G, sph, lim, m1.FP64, 1.0
    out, axis, per = m1.BC_OUTFLOW, m1.BC_AXIS, m1.BC_PERIODIC
    d.bc_lo[:] = [m1.BC_INFLOW, axis, per] if sph else [out] * 3
    d.bc_hi[:] = [out, axis, per] if sph else [out] * 3
    assert (fn(ctypes.byref(d), 256).nblocks > 0) == bool(fast)
