"""Group kernels (16 elements per work-group) against the plain kernels in FP64.

FP64 at orders 3..6 and FP32 at orders 3..7 (ranges below mc_min) on a
ragged box (a last group of 8 elements) with three clusters, whose ranges
begin and end inside groups, faces towards finer and coarser neighbours, a
gravity surface and jittered elements; and on a box with a fault, whose
elements store their derivatives.

Tolerance: a value is the end of sums of at most 8 B terms per step (volume,
traces and lifts of predictor and corrector), so after n steps two summation
orders differ by at most 8 B n unit roundoffs of the largest value of its kind
(stress or velocity).
"""
import numpy as np
import pytest

from paper_2107_06640_amd import inputs

pytestmark = pytest.mark.gpu

ZN = np.array([0.0, 0.5, 0.75, 0.875, 1.0]) * 1000.0 - 1000.0
STEPS = 2


def boxes():
    lts = inputs.coupled_box(3, 7, 4, cell=500.0, water_layers=1, z_nodes=ZN, jitter=0.1, seed=4)
    fault = inputs.fault_box(4, 4, 4, cell=500.0, k_fault=2, jitter=0.1, seed=3)
    return {"lts": (lts, 4), "fault": (fault, 1)}


def run(box, clusters, order, precision, kernel, **kw):
    from paper_2107_06640_amd import seis
    mesh, mats = box
    s = seis.from_mesh(mesh, mats, order, precision=precision, kernel=kernel, max_clusters=clusters, **kw)
    try:
        q = inputs.random_dofs(mesh.n_elements, s.B, seed=8, acoustic=mats[2] == 0)
        eta = np.random.default_rng(9).standard_normal((s.n_gravity_faces, s.nq)) * 0.1
        s.write(q, eta)
        s.run(STEPS)
        return s.read(), s.info()["n_clusters"]
    finally:
        s.close()


@pytest.mark.parametrize("name", ["lts", "fault"])
@pytest.mark.parametrize("precision,order", [("fp64", o) for o in (3, 4, 5, 6)] + [("fp32", o) for o in (3, 4, 5, 6, 7)])
def test_group_matches_plain(name, precision, order):
    box, clusters = boxes()[name]
    mesh, _ = box
    assert name == "fault" or mesh.n_elements % 16 != 0
    (q0, e0), _ = run(box, clusters, order, "fp64", "plain")
    (q1, e1), n = run(box, clusters, order, precision, "tuned", mc_min=mesh.n_elements + 1)
    assert name == "fault" or n >= 3
    B = q0.shape[1]
    u = 2.0**-53 if precision == "fp64" else 2.0**-24
    tol = 8 * B * STEPS * 2 ** (n - 1) * u  # the finest cluster's steps
    for part in (slice(0, 6), slice(6, 9)):
        err = np.abs(q1[:, :, part] - q0[:, :, part]).max() / np.abs(q0[:, :, part]).max()
        print(f"case: {name} {precision} order {order} rel {err:.1e} bound {tol:.1e}", flush=True)
        assert err <= tol
    if e0.size:
        assert np.abs(e1 - e0).max() <= tol * np.abs(e0).max()
