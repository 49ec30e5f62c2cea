"""Limited RK3 steps on mixed degrees whose workgroups hold several elements of
one degree, every one with another state along x: the limited stage rewrites
the rows of the volume buffer for the moments, at another stride, right after
the nodes have taken their derivatives from it."""
import numpy as np
import pytest

from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu
NE, SR, MHD = 0, 1, 2


@pytest.fixture(scope="module")
def dg():
    import torch
    assert torch.cuda.is_available()
    from paper_1609_00098_amd import dgmi
    return dgmi


# SR degree 4 (four elements per workgroup) is the form whose rows overlap;
# the others have one row layout, or the lane-per-node volume term
@pytest.mark.parametrize("system,N", [(SR, 4), (SR, 3), (SR, 5), (NE, 4), (MHD, 3), (MHD, 4)])
@pytest.mark.parametrize("flux", ["llf", "hll"])
def test_limited_step_full_groups(ora, dg, system, N, flux):
    """One limited step of 96 elements, all but eight of degree N (the last
    workgroup partly filled), against the oracle: 4e-12 dt max|L| (the mixed
    operator's bound through the stages) + 1e-13 max|U| (the limiter's)."""
    g = 4.0 / 3.0 if system else 5.0 / 3.0
    nel = (24, 2, 2)
    deg = np.full(96, N, dtype=np.int32)
    deg[5::13] = 2
    lim = "muscl"
    m = ora.mesh(system, nel, 2, g, kappa=0.5, limiter=lim, flux=flux)
    x = ora.mixed_node_coords(m, deg)[0]
    c = np.random.default_rng(7).uniform(0.3, 1.0, size=4)
    # smooth and monotone but for one drop: no decision rests on rounding
    drop, one = x > 0.37, np.ones_like(x)
    prim = np.stack([np.exp(c[0] * x) * np.where(drop, 0.3, 1.0), 0.2 * np.exp(-c[1] * x), 0.1 * one, 0.05 * one,
                     np.exp(c[2] * x) * np.where(drop, 0.2, 1.0)])
    mag = np.stack([one, 0.3 * np.exp(c[3] * x), 0.1 * one, 0.0 * one]) if system == MHD else None
    U, _, _ = ora.limit_mixed(m, deg, ora.prim2cons(system, g, prim, mag))
    L, P, nf = ora.rhs_mixed(m, deg, U)
    assert nf == 0
    dt = 1e-3 / float(max(np.abs(L[0] / U[0]).max(), np.abs(L[4] / U[4]).max()))
    Uo, nf = ora.step_mixed(m, deg, U, dt)
    assert nf == 0
    mesh = dg.Mesh(system, nel, 0, g, kappa=0.5, degrees=deg, flags=dg.FLAG_HLL if flux == "hll" else 0)
    dg.dgmi_set_limiter(mesh, dg.LIMITER_MUSCL, 0.0)
    Ud, Pd = to_dev(U), to_dev(P)
    dg.dg_step(mesh, Ud, Pd, dt)
    assert dg.dgmi_limited(mesh) > 0
    assert dg.dgmi_failures(mesh) == 0
    diff = np.abs(to_host(Ud) - Uo).max()
    assert diff <= 4e-12 * dt * np.abs(L).max() + 1e-13 * np.abs(U).max()
