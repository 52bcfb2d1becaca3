"""fornax_m1_step_noalloc on 2-D grids whose Runge-Kutta stage fills the static scratch up to the diagnostics
partials of about a thousand blocks: accepted, with the results of fornax_m1_step, however the
step kernel is tiled for speed."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _room(m1, nx, ny, G, prec):
    """Bytes left beside the stage and the partials of the largest power of two of planes per block (32
    to 4) with 1024 (double) or 2048 (float) blocks, all groups of a column in one block."""
    gb = 1
    while gb < 4 and G % (2 * gb) == 0:
        gb *= 2
    ntx = -(-nx // (64 // gb - 2))
    tm = 32
    while tm > 4 and ntx * -(-ny // tm) < (1024 if prec == 0 else 2048):
        tm //= 2
    nb = ntx * -(-ny // tm)
    al = lambda x: (x + 255) & ~255
    return m1.NOALLOC_SCRATCH_BYTES - 2 * al(8 * nb) - 2 * al(4 * nb) - al(3 * nx * ny * G * (8 if prec == 0 else 4))


@pytest.mark.parametrize("nx,G,prec", [(806, 1, 0), (806, 1, 1), (400, 2, 0), (440, 6, 1), (300, 4, 0), (1500, 2, 1)])
def test_largest_grid_of_the_static_scratch(nx, G, prec):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1806_07390_amd import m1
    ny = max(n for n in range(4, 4000) if _room(m1, nx, n, G, prec) >= 0)
    for n in (ny, ny - 1):
        ctx = m1.Context(m1.Config(ndim=2, n=(nx, n), G=G, precision=prec, integrator=m1.SSPRK2))
        torch.manual_seed(n)
        r = lambda: torch.rand(ctx.shape, dtype=ctx.dtype, device="cuda")
        E = 0.2 + r()
        F = [0.3 * E * (r() - 0.5), 0.3 * E * (r() - 0.5)]
        k, s, B, dt = 5 * r(), r(), r(), ctx.max_dt(0.4)
        d0, d1 = ctx.new_diag(), ctx.new_diag()
        ref = ctx.step(E, F, k, s, B, dt, diag=d0)
        got = ctx.step(E, F, k, s, B, dt, diag=d1, noalloc=True)
        torch.cuda.synchronize()
        assert torch.equal(ref[0], got[0]) and all(torch.equal(a, b) for a, b in zip(ref[1], got[1]))
        for key in d0:
            assert torch.equal(d0[key], d1[key])
