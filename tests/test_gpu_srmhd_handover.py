"""SRMHD stages hand the next one two primitive rows, from which it rebuilds the
five that the recovery returned.  Steps at a size where the operator's part of
the bound is the larger one, with both fluxes, and a node whose recovery fails:
it is at rest for its neighbours, as the five rows have it."""
import numpy as np
import pytest

from paper_1609_00098_amd import synth
from tests.gpu_util import normwise_err, to_dev, to_host

pytestmark = pytest.mark.gpu
MHD, GAMMA = 2, 4.0 / 3.0
LO, HI = (-0.2, 0.1, 0.0), (0.8, 1.3, 0.7)


@pytest.fixture(scope="module")
def dg():
    import torch
    assert torch.cuda.is_available()
    from paper_1609_00098_amd import dgmi
    return dgmi


def _state(ora, xyz, seed):
    unit = (xyz - np.array(LO)[:, None]) / (np.array(HI) - np.array(LO))[:, None]
    prim = synth.fourier_random_prims(unit, seed=seed, w_max=2.0, rho_range=(0.5, 2.0), p_range=(0.5, 2.0))
    rng = np.random.default_rng(seed)
    prim[[0, 4]] *= 1.0 + 0.002 * rng.uniform(-1.0, 1.0, (2, prim.shape[1]))  # the two sides of a face differ
    mag = 0.3 * np.stack([np.sin(2 * np.pi * (rng.integers(1, 3, size=3) @ unit) + c) for c in range(4)])
    mag[0] += 1.0
    return ora.prim2cons(MHD, GAMMA, prim, mag), prim


@pytest.mark.parametrize("nel", [(3, 1, 1), (3, 3, 1)])
@pytest.mark.parametrize("N", [1, 3, 4, 5])
@pytest.mark.parametrize("faces", ["periodic", "fixed"])
@pytest.mark.parametrize("flux", ["llf", "hll"])
def test_step(ora, dg, N, nel, faces, flux):
    """One step that changes U by 1e-3 of its size: 2e-12 dt max|L| (the
    operator bound through the stages) + 8 ulp max|U| (the combinations)."""
    lo, hi = [1.0, 0.1, -0.2, 0.05, 1.0, 0.5, 0.2, -0.1, 0.03], [0.7, -0.1, 0.3, 0.2, 2.0, 0.4, -0.2, 0.3, -0.05]
    bc = {0: (tuple(lo), tuple(hi))} if faces == "fixed" else None
    m = ora.mesh(MHD, nel, N, GAMMA, lo=LO, hi=HI, kappa=0.5, bc=bc, flux=flux)
    G = dg.Mesh(MHD, nel, N, GAMMA, lo=LO, hi=HI, kappa=0.5, flags=dg.FLAG_HLL if flux == "hll" else 0)
    if bc:
        dg.dgmi_set_boundary(G, 0, lo, hi)
    U, prim = _state(ora, ora.node_coords(m), seed=3 + N)
    L, _, nf = ora.rhs(m, U)
    assert nf == 0
    dt = 1e-3 * np.abs(U).max() / np.abs(L).max()
    Uo, nf = ora.step(m, U, dt)
    assert nf == 0
    Ud, Pd = to_dev(U), to_dev(prim)
    dg.dg_step(G, Ud, Pd, dt)
    assert dg.dgmi_failures(G) == 0
    assert np.abs(to_host(Ud) - Uo).max() <= 2e-12 * dt * np.abs(L).max() + 8 * 2.0 ** -52 * np.abs(U).max()
    _, Po, _ = ora.rhs(m, to_host(Ud))
    assert np.all(normwise_err(to_host(Pd), Po) <= 1e-12)


@pytest.mark.parametrize("N", [1, 3, 5])
@pytest.mark.parametrize("flux", ["llf", "hll"])
def test_failed_node_is_at_rest(ora, dg, N, flux):
    """tau below B^2/2 - D at one corner node: no bracket, the recovery returns
    the state at rest.  The neighbours' new states agree with those of a mixed
    mesh of equal degrees, whose stages keep all five rows, to 1e-12 of the
    step's change + 8 ulp (the same formulas, other instruction orders)."""
    nel = (3, 2, 2)
    flags = dg.FLAG_HLL if flux == "hll" else 0
    m = ora.mesh(MHD, nel, N, GAMMA, lo=LO, hi=HI, kappa=0.5, flux=flux)
    U, prim = _state(ora, ora.node_coords(m), seed=11)
    L, _, nf = ora.rhs(m, U)
    assert nf == 0
    dt = 1e-3 * np.abs(U).max() / np.abs(L).max()
    k = (N + 1) ** 3 * 4 + N  # a corner of an inner element
    BB = (U[5:8, k] ** 2).sum()
    U[0, k] = 0.1
    U[1:4, k] = [0.3, -0.2, 0.1]
    U[4, k] = 0.5 * BB - 0.5
    prim[:, k] = [U[0, k], 0.0, 0.0, 0.0, (GAMMA - 1.0) * (U[4, k] - 0.5 * BB)]
    out = []
    for mesh in (dg.Mesh(MHD, nel, N, GAMMA, lo=LO, hi=HI, kappa=0.5, flags=flags),
                 dg.Mesh(MHD, nel, 0, GAMMA, lo=LO, hi=HI, kappa=0.5, flags=flags,
                         degrees=np.full(12, N, dtype=np.int32))):
        Ud, Pd = to_dev(U), to_dev(prim)
        dg.dg_step(mesh, Ud, Pd, dt)
        assert dg.dgmi_failures(mesh) > 0
        out.append(to_host(Ud))
    change = np.abs(out[1] - U).max()
    assert np.isfinite(out[1]).all()
    assert np.abs(out[0] - out[1]).max() <= 1e-12 * change + 8 * 2.0 ** -52 * np.abs(U).max()
