"""Infinities and NaN in an activation reach exactly the points that the general products take them to.

The fused stages pad their products with zero rows and columns; a zero of the padding times an
infinity must not come back as NaN in a point's result. Networks whose sizes are no
multiple of a tile, against the same network on the chains of general products: the same points
are non-finite, with the same kind of value, and all others are equal bit for bit.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(5, 9), (16, 33), (33, 129), (48, 250), (32, 128)])
def test_projection_of_an_infinite_value(W, H):
    """Positive weights: an infinite channel value gives an infinite result, a NaN a NaN."""
    from paper_2107_06640_amd.fno import Kernels
    k, n = Kernels(), 517
    g = torch.Generator(device="cuda:0").manual_seed(1)
    Q1, Q2 = (0.1 + torch.rand(s, device="cuda:0", generator=g) for s in ((H, W), (1, H)))
    q1, q2 = torch.rand(H, device="cuda:0", generator=g), torch.rand(1, device="cuda:0", generator=g)
    v = torch.randn(W, n, device="cuda:0", generator=g)
    clean = torch.empty(n, device="cuda:0")
    k.head(n, W, H, Q1, q1, Q2, q2, v, clean)
    v[W - 1, 3] = float("inf")
    v[0, n - 1] = float("inf")
    v[0, 130] = float("nan")
    y = torch.empty(n, device="cuda:0")
    k.head(n, W, H, Q1, q1, Q2, q2, v, y)
    torch.cuda.synchronize()
    assert torch.isfinite(clean).all()
    assert torch.isposinf(y[[3, n - 1]]).all() and torch.isnan(y[130])
    rest = torch.ones(n, dtype=torch.bool, device="cuda:0")
    rest[[3, n - 1, 130]] = False
    assert torch.equal(y[rest], clean[rest])


@pytest.mark.parametrize("W,H", [(5, 9), (16, 33), (33, 129), (48, 250), (32, 128)])
def test_projection_gradient_of_an_infinite_value(W, H):
    """Positive weights and values: an infinite gradient stays one at its point, and in every weight's sum."""
    from paper_2107_06640_amd.fno import Kernels
    k, n = Kernels(), 517
    g = torch.Generator(device="cuda:0").manual_seed(2)
    rand = lambda *s: 0.1 + torch.rand(*s, device="cuda:0", generator=g)
    Q1, Q2, q1, v, dy = rand(H, W), rand(1, H), rand(H), rand(W, n), rand(n)
    out = []
    for bad in (False, True):
        if bad:
            dy[[2, n - 1]] = float("inf")
        r = [torch.empty(s, device="cuda:0") for s in ((W, n), (H, W), (H,), (1, H))]
        k.head_backward(n, W, H, Q1, q1, Q2, v, dy, *r)
        out.append(r)
    torch.cuda.synchronize()
    clean, got = out
    assert all(torch.isfinite(t).all() for t in clean)
    rest = torch.ones(n, dtype=torch.bool, device="cuda:0")
    rest[[2, n - 1]] = False
    assert torch.isposinf(got[0][:, ~rest]).all() and torch.equal(got[0][:, rest], clean[0][:, rest])
    assert all(torch.isposinf(t).all() for t in got[1:])


@pytest.mark.parametrize("shape", [(9, 17, 7, 2, 5, 9), (12, 12, 8, 3, 16, 33), (25, 33, 31, 12, 33, 129)])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_network_keeps_the_kind_of_every_value(shape, value):
    """A non-finite input spreads through the spectral layers to its sample, not to the others."""
    from paper_2107_06640_amd.fno import FNO
    X, Y, T, m, W, H = shape
    nets = [FNO(X, Y, T, cin=3, width=W, modes=m, layers=2, hidden=H, seed=3) for _ in range(2)]
    assert nets[0].fused
    nets[1].fused = False
    g = torch.Generator(device="cuda:0").manual_seed(5)
    u = torch.randn(3, 3, X, Y, T, device="cuda:0", generator=g)
    u[1, 1, X // 2, Y // 3, T - 1] = value
    a, b = (net.forward(u) for net in nets)
    torch.cuda.synchronize()
    for sample in (0, 2):
        assert torch.isfinite(a[:, sample]).all()
    assert torch.equal(torch.nan_to_num(a, 0.0, 1.0, -1.0), torch.nan_to_num(b, 0.0, 1.0, -1.0))
    assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.isinf(a), torch.isinf(b))
