"""Which kernels a launch takes, and launches of different kernels handing over to each other.

The box of 9180 elements has clusters of 1532, 2054 and 5594, so a launch
covers 1532, 3586 or 9180 elements, or with a launch per cluster starts at 1532 or
3586, inside a group of 16 (whose half-step integrals two launches then write).
FP64, and FP32 with mc_min beyond the box, run every one of them on the group
kernels; mc_min of 2048 and 4000 give the larger ones to the wavefront kernels, so
that the faces between clusters hand over from either form to the other, in both
directions and within the pair of steps of a coarser neighbour.

Tolerances against the plain FP64 kernels. FP64: as in test_gpu_group.py, 8 B n unit
roundoffs of the largest value of a kind after n steps. FP32: every one of n steps rounds a
value some 8 B times, independently, so the relative L2 error of a kind is about
sqrt(8 B n) roundoffs of at most half a unit each: sqrt(8 B n) 2^-24.

Below 256 elements every launch takes the plain kernels: the same bits as a handle that
asks for them.
"""
import functools

import numpy as np
import pytest

from paper_2107_06640_amd import inputs

pytestmark = pytest.mark.gpu

ZN = np.array([0.0, 0.5, 0.75, 0.875, 0.9375, 0.96875, 1.0]) * 1000.0 - 1000.0
CLUSTERS = [1532, 2054, 5594]
STEPS = 2


@functools.lru_cache(maxsize=1)
def box():
    return inputs.coupled_box(15, 17, 6, cell=500.0, water_layers=1, z_nodes=ZN, jitter=0.1, seed=4)


def run(mesh, mats, order, precision, kernel, **kw):
    from paper_2107_06640_amd import seis
    s = seis.from_mesh(mesh, mats, order, precision=precision, kernel=kernel, max_clusters=3, **kw)
    try:
        q = inputs.random_dofs(mesh.n_elements, s.B, seed=8, acoustic=mats[2] == 0)
        eta = np.random.default_rng(9).standard_normal((s.n_gravity_faces, s.nq)) * 0.1
        s.write(q, eta)
        s.run(STEPS)
        return *s.read(), s.info()["cluster_size"]
    finally:
        s.close()


@functools.lru_cache(maxsize=1)
def reference(order):
    q, e, n = run(*box(), order, "fp64", "plain")
    assert n == CLUSTERS and CLUSTERS[0] % 16 and (CLUSTERS[0] + CLUSTERS[1]) % 16
    return q, e


CASES = [(o, "fp64", None) for o in (3, 4, 5, 6)] + [(o, "fp32", m) for o in (3, 4, 5, 6, 7) for m in (2048, 4000, 10000)]


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("order,precision,mc_min", sorted(CASES, key=lambda c: c[0]))
def test_ranges_hand_over_to_each_other(order, precision, mc_min, fused):
    q0, e0 = reference(order)
    q1, e1, _ = run(*box(), order, precision, "tuned", mc_min=mc_min, fused=fused)
    terms = 8 * q0.shape[1] * STEPS * 2 ** (len(CLUSTERS) - 1)
    for part in (slice(0, 6), slice(6, 9)):
        a, b = q1[:, :, part], q0[:, :, part]
        if precision == "fp64":
            err, tol = np.abs(a - b).max() / np.abs(b).max(), terms * 2.0**-53
        else:
            err, tol = np.sqrt(((a - b) ** 2).sum() / (b ** 2).sum()), np.sqrt(terms) * 2.0**-24
        print(f"case: {precision} order {order} mc_min {mc_min} fused {fused} rel {err:.1e} bound {tol:.1e}", flush=True)
        assert err <= tol
    assert np.abs(e1 - e0).max() <= tol * np.abs(e0).max()


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("precision,order", [("fp64", o) for o in (3, 4, 5, 6)] + [("fp32", o) for o in (3, 5, 7)])
def test_small_ranges_are_the_plain_kernels(precision, order, fused):
    mesh, mats = inputs.coupled_box(3, 3, 3, cell=500.0, water_layers=1, jitter=0.1, seed=4)
    a = run(mesh, mats, order, precision, "tuned", fused=fused)
    b = run(mesh, mats, order, precision, "plain", fused=fused)
    assert sum(a[2]) < 256 and len(a[2]) == 3
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
