"""The counting kernels' operations and bytes against a count by hand (host logic, no launches).

The library is a stub that accepts every call, so a network on the CPU only sequences its stages.
"""
import pytest
import torch

from paper_2107_06640_amd import fno


class AcceptAll:
    """fno_*(...) -> 0; every shape fits the fused stages."""

    def __getattr__(self, name):
        return lambda *a: 1 if name == "fno_fused_shape" else 0


@pytest.fixture
def kernels(monkeypatch):
    monkeypatch.setattr(fno, "_lib", AcceptAll)
    return fno.CountingKernels()


def test_one_training_step(kernels):
    X, Y, T, C, W, m, L, H, B = 10, 12, 8, 3, 5, 2, 3, 7, 2
    net = fno.FNO(X, Y, T, cin=C, width=W, modes=m, layers=L, hidden=H, device="cpu", kernels=kernels)
    assert net.fused
    y = net.forward(torch.zeros(C, B, X, Y, T), keep=True)
    net.backward(torch.zeros_like(y))
    S, m2 = B * X * Y * T, 2 * m
    nm = m2 * m2 * m
    act = W * S                              # an activation
    ty, x0 = W * B * X * 2 * m2 * m, W * B * 2 * nm  # spectra along t and y, and along x too
    x_in, x_out = W * B * X * 2 * m2 * m, W * B * 2 * nm
    mix = 4 * B * W * nm + 2 * W * W * nm    # in, out (re, im) and R
    forward = S * (C + W) + S * (W + 1)      # lift, projection
    for l in range(L):
        last = l == L - 1
        forward += act + ty                  # t and y: activation in, spectrum out
        forward += x_in + x_out + mix + x_out + x_in
        forward += ty + act + (1 if last else 2) * act  # spectrum and input in; z, and gelu(z) between layers, out
    backward = S * (2 * W + 1)               # projection: v and dy in, dv out
    for l in range(L):
        backward += S * (2 * W if l == L - 1 else 4 * W)  # dz (or da, z, dz) and x
        backward += act + ty + x_in + x_out + 2 * mix + x_out + x_in
        backward += ty + act + act
    backward += S * (W + C)                  # lift: dz and u
    assert x0 == x_out
    assert kernels.bytes == 4 * (forward + backward)
    assert kernels.calls == 2 + 5 * L + 2 + 7 * L


def test_one_inference(kernels):
    X, Y, T, C, W, m, H = 6, 9, 5, 2, 4, 1, 6
    net = fno.FNO(X, Y, T, cin=C, width=W, modes=m, layers=1, hidden=H, device="cpu", kernels=kernels)
    net.forward(torch.zeros(C, 1, X, Y, T))
    S, K = X * Y * T, 4 * m
    assert kernels.flops == 2 * (S * C * W + W * X * (Y * 2 * m * T + 2 * K * m * Y) + W * 2 * K * X * 2 * m * m
                                 + 4 * (4 * m ** 3) * W * W + W * 2 * X * K * 2 * m * m
                                 + S * W * (W + 2 * m) + X * W * Y * 2 * m * K + S * H * (W + 1))
