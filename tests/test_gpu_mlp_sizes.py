"""The network's kernels at the sizes where their work split changes: below
and beyond one workgroup, at tile edges, in column slices of a wider matrix."""
import numpy as np
import pytest

from oracle import mlp as M
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import torch
    assert torch.cuda.is_available()
    from paper_1609_00098_amd import dgmi
    return dgmi


# one workgroup up to 1024 samples, 512 workgroups from 523,265 on
@pytest.mark.parametrize("n", [2, 63, 257, 1024, 1025, 40_003, 523_264, 524_289])
def test_normalization_sizes(dg, n):
    """Means and deviations against FP64.  The sums are FP64, so the mean is
    the exact one rounded to FP32 (2^-24 relative) and the variance carries
    n 2^-53 of E[x^2], at most 1e-9 of it here (|mean| <= 10 sd): 2e-7
    relative covers both."""
    import torch
    rng = np.random.default_rng(n)
    wide = torch.zeros((5, n + 7), dtype=torch.float32, device="cuda")
    x = (rng.normal(size=(5, n)) * np.array([[1.0], [0.1], [3.0], [1e-3], [20.0]]) + np.array([[1.0], [1.0], [-2.0], [0.01], [5.0]]))
    x = x.astype(np.float32)
    t = rng.normal(size=n).astype(np.float32)
    wide[:, 3:3 + n] = to_dev(x)
    net = dg.Mlp(seed=1)
    before = to_host(dg.mlp_get(net))
    dg.mlp_fit_normalization(net, wide[:, 3:3 + n], to_dev(t))
    p = to_host(dg.mlp_get(net)).astype(np.float64)
    assert np.array_equal(p[:M.NW], before[:M.NW])
    c = np.concatenate([x, t[None]]).astype(np.float64)
    mean, sd = c.mean(1), c.std(1)
    got_mean, got_sd = np.append(p[M.O_MU:M.O_MU + 5], p[M.O_YMU]), np.append(p[M.O_SD:M.O_SD + 5], p[M.O_YSD])
    assert np.all(np.abs(got_mean - mean) <= 2e-7 * np.abs(mean) + 1e-12 * sd)
    assert np.all(np.abs(got_sd - sd) <= 2e-7 * sd)
