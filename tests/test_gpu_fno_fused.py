"""The network's fused stages against its chains of general products on the GPU.

Both round the same operands to BF16 and accumulate the same K steps in FP32,
so outputs equal bit for bit. Weight gradients are sums over all points in
another order: with n terms of FP32 the two orders differ by at most about
sqrt(n) 2^-24 of the root of the sum of squares, which 2e-5 of the gradient's
norm covers for the sizes here. Sizes sit at the edges of the tiles: grids
that are no multiple of 4, 16 or 32 points, one and more 16-row tiles of every
matrix, one and two 32-wide K steps.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

SHAPES = [
    # X, Y, T, modes, batch, cin, width, hidden, layers
    (16, 12, 8, 3, 3, 3, 8, 16, 3),      # one tile of everything, T a multiple of 4
    (9, 17, 7, 2, 1, 2, 5, 9, 2),        # odd everywhere: scalar loads, partial tiles
    (24, 32, 32, 12, 2, 4, 32, 128, 2),  # the surrogate's width, modes and hidden size
    (25, 33, 31, 12, 1, 4, 33, 129, 1),  # one past a tile: two K steps of the width, two hidden blocks
    (33, 40, 33, 16, 17, 5, 16, 33, 1),  # most modes, two K steps along t, a second batch tile
    (12, 9, 16, 4, 2, 17, 48, 256, 2),   # the widest network
]


def pair(shape):
    from paper_2107_06640_amd.fno import FNO
    X, Y, T, m, B, cin, W, H, L = shape
    nets = [FNO(X, Y, T, cin=cin, width=W, modes=m, layers=L, hidden=H, seed=3) for _ in range(2)]
    assert nets[0].fused
    nets[1].fused = False
    g = torch.Generator(device="cuda:0").manual_seed(5)
    for k, v in nets[0].params.items():
        if v.ndim == 1:
            v.copy_(0.1 * torch.randn(v.shape, device="cuda:0", generator=g))
        nets[1].params[k].copy_(v)
    u = torch.randn(cin, B, X, Y, T, device="cuda:0", generator=g)
    y = torch.randn(1, B, X, Y, T, device="cuda:0", generator=g)
    return nets, u, y


@pytest.mark.parametrize("shape", SHAPES)
def test_fused_network_equals_the_chain_of_products(shape):
    nets, u, y = pair(shape)
    plain = nets[0].forward(u)
    outs, grads = [], []
    for net in nets:
        out = net.forward(u, keep=True)
        _, dy = net.loss(out, y)
        for g in net.grads.values():
            g.fill_(float("nan"))  # every gradient is overwritten
        grads.append({k: v.clone() for k, v in net.backward(dy).items()})
        outs.append(out.clone())
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])
    assert torch.equal(plain, outs[1])  # without keeping activations
    for k, want in grads[1].items():
        err = (grads[0][k] - want).double().norm() / want.double().norm()
        assert err < 2e-5, (k, float(err))


def test_shapes_beyond_the_fused_stages_take_the_general_products():
    from paper_2107_06640_amd.fno import FNO, Kernels
    k = Kernels()
    assert k.fused_shape(128, 128, 64, 48, 4, 16, 256)
    for bad in ((129, 8, 8, 1, 4, 2, 8), (8, 8, 65, 1, 4, 2, 8), (8, 8, 8, 49, 4, 2, 8), (8, 8, 8, 1, 49, 2, 8),
                (64, 64, 64, 1, 4, 17, 8), (8, 8, 8, 1, 4, 2, 257)):
        assert not k.fused_shape(*bad)
    net = FNO(8, 8, 8, cin=2, width=50, modes=2, layers=1, hidden=8, seed=0)
    assert not net.fused
    y = net.forward(torch.randn(2, 1, 8, 8, 8, device="cuda:0"))
    torch.cuda.synchronize()
    assert torch.isfinite(y).all()
