"""mlp_forward's activation to the end of the exponential's FP32 range."""
import pytest

pytestmark = pytest.mark.gpu


def test_activation_tails():
    """A network with one path, y = silu(2^100 silu(x)), against FP64.  Relative
    bar: below -80 half a spacing of the subnormal bfloat16 parts of the inner
    activation (4.6e-41 of 2.6e-37: 1.8e-4) twice over; above, where the outer one
    is linear or its argument below 1, a few ulp of the exponential's argument
    (128 at most: 8e-6) times the derivative's weight."""
    import torch
    from paper_1609_00098_amd import dgmi as dg
    q = torch.zeros(4621, device="cuda")
    q[0], q[384], q[4480 + 64] = 1.0, 2.0 ** 100, 1.0  # W1[0][0], W2[0][0], W3[0]
    q[4614:4619] = 1.0  # deviations
    q[4620] = 1.0
    net = dg.Mlp(seed=1)
    dg.mlp_set(net, q)
    v = torch.tensor([-88.7, -88.5, -88.0, -87.4, -86.0, -83.0, -80.0, -1e-30, 0.0, 1e-30], device="cuda")
    x = torch.zeros(5, len(v), device="cuda")
    x[0] = v
    y = dg.mlp_forward(net, x).double()
    s = v.double() / (1 + torch.exp(-v.double())) * 2.0 ** 100
    e = s / (1 + torch.exp(-s))
    assert (y - e).abs().le(4e-4 * e.abs()).all()
