"""The recovery compiled per mode: tolerance and polish, every seed, states from
weakly to strongly magnetised, points that need the bisection's many steps, and
unphysical ones, at sizes around a wave and a workgroup.

Bars: tolerance mode, backward residual <= 1e-10 at every point; polish mode,
primitives within 1e-12 of the oracle (norm-wise); failure flags as
constructed."""
import numpy as np
import pytest

from paper_1609_00098_amd import synth
from tests.gpu_util import normwise_err, to_dev, to_host

pytestmark = pytest.mark.gpu
SR, MHD = 1, 2
G43 = 4.0 / 3.0


@pytest.fixture(scope="module")
def dg():
    import torch
    assert torch.cuda.is_available()
    from paper_1609_00098_amd import dgmi
    return dgmi


def _states(system, n, seed, sigma):
    if system == SR:
        return synth.sr_samples(n, seed=seed), None
    return synth.srmhd_samples(n, seed=seed, sigma_range=sigma)


@pytest.mark.parametrize("system,sigma", [(SR, None), (MHD, (1e-4, 1e-2)), (MHD, (1.0, 10.0)), (MHD, (50.0, 200.0))])
@pytest.mark.parametrize("n", [1, 65, 1000, 20_001])
def test_tolerance_mode_every_seed(ora, dg, system, sigma, n):
    import torch
    prim, mag = _states(system, n, n, sigma)
    U = ora.prim2cons(system, G43, prim, mag)
    Ud = to_dev(U)
    for guess in (dg.GUESS_INPUT, dg.GUESS_PLAIN, dg.GUESS_F0):
        P = to_dev(prim * 1.3)
        it = torch.zeros(n, dtype=torch.uint8, device="cuda")
        fl = torch.full((n,), 7, dtype=torch.uint8, device="cuda")
        dg.con2prim(system, G43, Ud, P, guess=guess, tol=1e-10, iters_out=it, fail_out=fl)
        assert int(fl.sum()) == 0 and int(it.min()) >= 1
        assert ora.backward_residual(system, G43, U, to_host(P)).max() <= 1e-10


@pytest.mark.parametrize("system,sigma", [(SR, None), (MHD, (1e-4, 1e-2)), (MHD, (1.0, 10.0))])
@pytest.mark.parametrize("guess", ["input", "plain", "f0"])
def test_polish_mode_every_seed(ora, dg, system, sigma, guess):
    prim, mag = _states(system, 5001, 3, sigma)
    U = ora.prim2cons(system, G43, prim, mag)
    P = to_dev(prim * (1 + 1e-3))
    dg.con2prim(system, G43, to_dev(U), P, tol=0.0,
                guess={"input": dg.GUESS_INPUT, "plain": dg.GUESS_PLAIN, "f0": dg.GUESS_F0}[guess])
    Po, _, nf = ora.cons2prim(system, G43, U)
    assert nf == 0 and np.all(normwise_err(to_host(P), Po) <= 1e-12)


@pytest.mark.parametrize("system", [SR, MHD])
@pytest.mark.parametrize("tol", [0.0, 1e-10])
def test_unphysical_points_fail_alone(ora, dg, system, tol):
    """Negative density, negative energy, NaN and too much momentum fail and
    leave the points around them as they are without them."""
    import torch
    prim, mag = _states(system, 300, 9, (1e-2, 1.0))
    U = ora.prim2cons(system, G43, prim, mag)
    clean = torch.zeros((5, 300), dtype=torch.float64, device="cuda")
    dg.con2prim(system, G43, to_dev(U), clean, guess=dg.GUESS_F0, tol=tol)
    bad = [0, 63, 64, 201]
    V = U.copy()
    V[0, 0], V[4, 63], V[4, 64] = -1.0, -5.0, np.nan
    V[1:4, 201] *= 50.0
    P, fl = torch.zeros_like(clean), torch.zeros(300, dtype=torch.uint8, device="cuda")
    dg.con2prim(system, G43, to_dev(V), P, guess=dg.GUESS_F0, tol=tol, fail_out=fl)
    assert np.flatnonzero(to_host(fl)).tolist() == bad
    keep = np.setdiff1d(np.arange(300), bad)
    assert np.array_equal(to_host(P)[:, keep], to_host(clean)[:, keep])
