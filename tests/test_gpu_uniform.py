"""A uniform medium at rest without matter stays what it is, to the last bit: the two fluxes of a
zone in each direction are equal and cancel exactly, so E is kept and no flux component arises.
Three-dimensional Cartesian grids in double (rows of one, two and four x tiles, group counts that
leave rows idle), every limiter, both integrators, and the velocity step's transport at rest; the
y widths are such that dt/dy is not a power of two."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny", [9, 61, 75, 100])
@pytest.mark.parametrize("opts", ["minmod", "mc", "ppm-rk2", "m1", "velocity"])
@pytest.mark.parametrize("G", [1, 2, 5, 12])
def test_uniform_medium_at_rest(G, opts, ny):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1806_07390_amd import m1
    kw = {"mc": dict(limiter=m1.LIMITER_MC), "ppm-rk2": dict(limiter=m1.LIMITER_PPM, integrator=m1.SSPRK2),
          "m1": dict(wavespeed=m1.WAVESPEED_M1)}.get(opts, {})
    ctx = m1.Context(m1.Config(ndim=3, n=(19, ny, 14), G=G, bc_lo=(m1.BC_PERIODIC,) * 3, bc_hi=(m1.BC_PERIODIC,) * 3,
                               **kw))
    E0 = np.random.default_rng(ny).uniform(0.3, 3.0, G)
    E = torch.from_numpy(np.broadcast_to(E0, ctx.shape).copy()).cuda()
    F = [torch.zeros_like(E) for _ in range(3)]
    none = torch.zeros_like(E)
    dt = ctx.max_dt(0.37)
    U = (E, F)
    if opts == "velocity":
        ctx.set_group_edges(np.arange(1.0, G + 2.0))
        vf = [torch.zeros((3,) + ctx.face_shape(d), dtype=E.dtype, device="cuda") for d in range(3)]
    for _ in range(3):
        if opts == "velocity":
            U = ctx.step_velocity(U[0], U[1], none, none, none, vf, dt)
        else:
            U = ctx.step(U[0], U[1], none, none, none, dt)
    torch.cuda.synchronize()
    for f in U[1]:
        assert torch.count_nonzero(f) == 0
    assert torch.equal(U[0], E)
