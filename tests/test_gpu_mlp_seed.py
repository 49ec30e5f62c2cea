"""The learned seed is the network's output at the features that training uses,
also for states whose density lies at the ends of the FP32 range."""
import numpy as np
import pytest

from paper_1609_00098_amd import synth
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu
SR, MHD, G43 = 1, 2, 4.0 / 3.0


@pytest.mark.parametrize("system", [SR, MHD])
@pytest.mark.parametrize("scale", [1.0, 3e-39, 1e-30, 1e30])
def test_seed_is_the_networks(ora, system, scale):
    """The learned recovery takes one evaluation more (its f(0) feature) than
    one seeded by hand with D exp(mlp_forward(mlp_features)).  Both seeds carry
    FP32 rounding, 1e-7 of p or so, which moves a count only where a residual
    falls that close to the tolerance: at most 1 point in 1,000 may differ."""
    import torch
    from paper_1609_00098_amd import dgmi as dg
    n = 20_003
    prim, mag = (synth.sr_samples(n, seed=3), None) if system == SR else synth.srmhd_samples(n, seed=3)
    U = to_dev(ora.prim2cons(system, G43, prim, mag))
    net = dg.Mlp(seed=5)
    x, t = dg.mlp_features(system, G43, U, prim=to_dev(prim))
    dg.mlp_fit_normalization(net, x, t)
    dg.mlp_train(net, x, t, batch=1000, epochs=4, lr0=3e-3, lr1=1e-4)
    # a state scaled in its energies and, by the root, in its field
    U *= scale
    if system == MHD:
        U[5:] *= scale ** -0.5
    P, Q = torch.zeros((5, n), dtype=torch.float64, device="cuda"), torch.zeros((5, n), dtype=torch.float64, device="cuda")
    it, jt = torch.zeros(n, dtype=torch.uint8, device="cuda"), torch.zeros(n, dtype=torch.uint8, device="cuda")
    dg.con2prim(system, G43, U, P, guess=dg.GUESS_LEARNED, mlp=net, tol=1e-10, iters_out=it)
    x, _ = dg.mlp_features(system, G43, U, prim=P)
    Q[4] = U[0] * torch.exp(dg.mlp_forward(net, x).double())
    dg.con2prim(system, G43, U, Q, guess=dg.GUESS_INPUT, tol=1e-10, iters_out=jt)
    assert int((it != jt + 1).sum()) <= n // 1000
    assert np.isfinite(float(P.sum())) and float((P[4] - Q[4]).norm() / Q[4].norm()) <= 1e-8
