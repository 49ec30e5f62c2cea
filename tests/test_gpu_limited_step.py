"""The limiter's moment sums and decisions for the degrees, and the element
counts per workgroup, that its other tests leave out, and limited RK3 steps
whose intermediate stages keep only the rows the next one reads.

States vary along x only (smooth and monotone but for one drop), so that no
decision rests on rounding.  Bars: limited component counts equal, limited U
1e-13 norm-wise, primitives 1e-12; a step within 2e-12 dt max|L| + 8 ulp max|U|
(scales over all variables)."""
import numpy as np
import pytest

from tests.gpu_util import normwise_err, to_dev, to_host

pytestmark = pytest.mark.gpu
NE, SR, MHD = 0, 1, 2


@pytest.fixture(scope="module")
def dg():
    import torch
    assert torch.cuda.is_available()
    from paper_1609_00098_amd import dgmi
    return dgmi


def _pair(ora, dg, system, nel, N, lim):
    g = 4.0 / 3.0 if system else 1.4
    m = ora.mesh(system, nel, N, g, kappa=0.5, limiter=lim)
    G = dg.Mesh(system, nel, N, g, kappa=0.5)
    dg.dgmi_set_limiter(G, {"muscl": dg.LIMITER_MUSCL, "minmod": dg.LIMITER_MINMOD}[lim], 0.0)
    x = ora.node_coords(m)[0]
    c = np.random.default_rng(N + 10 * system).uniform(0.3, 1.0, size=5)
    drop, one = x > 0.37, np.ones_like(x)
    prim = np.stack([np.exp(c[0] * x) * np.where(drop, 0.3, 1.0), 0.2 * np.exp(-c[1] * x), 0.1 * one,
                     0.05 * np.exp(c[2] * x), np.exp(c[3] * x) * np.where(drop, 0.2, 1.0)])
    mag = np.stack([one, 0.3 * np.exp(c[4] * x), 0.1 * one, 0.0 * one]) if system == MHD else None
    return m, G, ora.prim2cons(system, g, prim, mag), prim


@pytest.mark.parametrize("system,N,lim", [(NE, 3, "muscl"), (NE, 4, "minmod"), (SR, 2, "minmod"), (SR, 4, "muscl"),
                                          (SR, 6, "minmod"), (SR, 7, "muscl"), (MHD, 2, "muscl"), (MHD, 4, "minmod"),
                                          (MHD, 5, "muscl"), (MHD, 7, "minmod")])
def test_limit_other_degrees(ora, dg, system, N, lim):
    m, G, U, prim = _pair(ora, dg, system, (7, 1, 3) if N <= 3 else (5, 1, 1), N, lim)
    Uo, count = ora.limit(m, U)
    assert count > 0
    Ud, Pd = to_dev(U), to_dev(prim * (1 + 1e-3))
    dg.dg_limit(G, Ud, Pd)
    assert dg.dgmi_limited(G) == count and dg.dgmi_failures(G) == 0
    assert np.all(normwise_err(to_host(Ud), Uo) <= 1e-13)
    Po, _, nf = ora.cons2prim(system, m.gamma, Uo)
    assert nf == 0 and np.all(normwise_err(to_host(Pd), Po) <= 1e-12)


@pytest.mark.parametrize("system,N", [(NE, 1), (NE, 4), (SR, 1), (SR, 2), (SR, 3), (SR, 5), (MHD, 1), (MHD, 3)])
def test_limited_step_keeps_needed_rows(ora, dg, system, N):
    m, G, U, prim = _pair(ora, dg, system, (7, 1, 3) if N <= 3 else (5, 1, 1), N, "muscl")
    L, _, nf = ora.rhs(m, U)
    assert nf == 0
    dt = 1e-4 * np.abs(U).max() / np.abs(L).max()
    Uo, nf = ora.step(m, U, dt)
    assert nf == 0
    Ud, Pd = to_dev(U), to_dev(prim)
    dg.dg_step(G, Ud, Pd, dt)
    assert dg.dgmi_failures(G) == 0
    assert np.abs(to_host(Ud) - Uo).max() <= 2e-12 * dt * np.abs(L).max() + 8 * 2.0 ** -52 * np.abs(U).max()
    Po, _, nf = ora.cons2prim(system, m.gamma, to_host(Ud))
    assert nf == 0 and np.all(normwise_err(to_host(Pd), Po) <= 1e-12)
