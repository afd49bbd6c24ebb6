"""The two forms of the sampling kernel: nine sums of a point in nine threads, or in one.

Large sets that follow the mesh take one thread per point, in FP64 larger ones
in any order, all others nine. Both sum the modes in ascending order, so a
point's values are the same bits in either form, whatever the set around it.
Sizes: around the 16 points that share a run of threads, the 4096 from which
work-groups are larger, and the 20 480 (mesh order) and 32 768 (FP64) from
which the second form runs. Scattered sets from 6144 on run the first form a mode
a trip, with the nine threads of a point side by side.
"""
import time

import numpy as np
import pytest

from paper_2107_06640_amd import inputs

pytestmark = pytest.mark.gpu

ORDERED, WIDE, SCATTERED = 20480, 32768, 6144


def sample(s, pts):
    import torch
    i = s.points(pts)
    out = torch.full((len(pts), 9), float("nan"), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    s.sample_into(i, out.data_ptr())
    s.sync()
    return out.cpu().numpy()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [1, 15, 17, 65, 4095, 4097, ORDERED - 1, ORDERED + 1, WIDE + 3])
def test_forms_agree_bit_for_bit(precision, n):
    from paper_2107_06640_amd import seis
    mesh, mats = inputs.coupled_box(4, 4, 5, cell=500.0, water_layers=2, jitter=0.1, seed=3)
    s = seis.from_mesh(mesh, mats, 5, precision=precision, kernel="plain")
    try:
        s.write(inputs.random_dofs(mesh.n_elements, s.B, seed=4, acoustic=mats[2] == 0))
        rng = np.random.default_rng(n)
        # mesh order: each element's points follow one another
        e = np.sort(rng.integers(0, mesh.n_elements, n))
        w = rng.dirichlet(np.full(4, 3.0), n)
        pts = np.einsum("nv,nvd->nd", w, mesh.xyz[mesh.tet[e]])
        got = sample(s, pts)
        perm = rng.permutation(n)
        mixed = sample(s, pts[perm])
        assert np.isfinite(got).all()
        assert np.array_equal(got[perm], mixed)
        pick = rng.choice(n, min(n, 40), replace=False)
        assert np.array_equal(got[pick], sample(s, pts[pick]))
    finally:
        s.close()


def test_scattered_receivers_share_the_chip():
    """256 scattered receivers are four wavefronts with a thread per point, each waiting for 64 rows of
    the state a load (15 times the call with 16 receivers); nine threads a point fill 36."""
    import torch
    from paper_2107_06640_amd import seis
    mesh, mats = inputs.coupled_box(16, 16, 12, cell=500.0, water_layers=3)
    s = seis.from_mesh(mesh, mats, 6, precision="fp32")
    try:
        s.write(inputs.random_dofs(mesh.n_elements, s.B, seed=4, acoustic=mats[2] == 0))
        rng = np.random.default_rng(1)
        lo, hi = mesh.xyz.min(axis=0), mesh.xyz.max(axis=0)
        took = []
        for n in (16, 256):
            i = s.points(rng.uniform(lo + 1.0, hi - 1.0, (n, 3)))
            out = torch.empty(n, 9, dtype=torch.float64, device="cuda")
            best = np.inf
            for _ in range(6):
                s.sync()
                t = time.perf_counter()
                for _ in range(100):
                    s.sample_into(i, out.data_ptr())
                s.sync()
                best = min(best, time.perf_counter() - t)
            took.append(best / 100)
        print(f"16 receivers {took[0] * 1e6:.1f} us, 256 receivers {took[1] * 1e6:.1f} us", flush=True)
        assert took[1] < 5 * took[0]
    finally:
        s.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [SCATTERED - 1, SCATTERED, SCATTERED + 1])
def test_scattered_order_agrees_bit_for_bit(precision, n):
    """Around the size from which scattered points run a mode a trip, their threads dense."""
    from paper_2107_06640_amd import seis
    mesh, mats = inputs.coupled_box(4, 4, 5, cell=500.0, water_layers=2, jitter=0.1, seed=3)
    for order in (2, 6):
        s = seis.from_mesh(mesh, mats, order, precision=precision, kernel="plain")
        try:
            s.write(inputs.random_dofs(mesh.n_elements, s.B, seed=4, acoustic=mats[2] == 0))
            rng = np.random.default_rng(n)
            e = rng.integers(0, mesh.n_elements, n)
            pts = np.einsum("nv,nvd->nd", rng.dirichlet(np.full(4, 3.0), n), mesh.xyz[mesh.tet[e]])
            got = sample(s, pts)
            assert np.isfinite(got).all()
            order_ = np.argsort(e, kind="stable")
            assert np.array_equal(got[order_], sample(s, pts[order_]))
            for r in range(0, n, 2048):
                assert np.array_equal(got[r:r + 2048], sample(s, pts[r:r + 2048]))
        finally:
            s.close()


def test_scattered_receivers_keep_their_rows():
    """16 384 scattered receivers in FP64 against 4096: four times the rows, of which many are in a cache
    by then. With eight modes in flight the wavefronts spread over the modes and rows leave it before they are shared
    (4.0 times the time at order 8, 2.5 with a mode a trip); the limit lies between the two."""
    import torch
    from paper_2107_06640_amd import seis
    mesh, mats = inputs.coupled_box(20, 20, 10, cell=500.0, water_layers=3)
    s = seis.from_mesh(mesh, mats, 8, precision="fp64", kernel="plain")
    try:
        rng = np.random.default_rng(1)
        lo, hi = mesh.xyz.min(axis=0), mesh.xyz.max(axis=0)
        took = []
        for n in (4096, 16384):
            i = s.points(rng.uniform(lo + 1.0, hi - 1.0, (n, 3)))
            out = torch.empty(n, 9, dtype=torch.float64, device="cuda")
            best = np.inf
            for _ in range(6):
                s.sync()
                t = time.perf_counter()
                for _ in range(20):
                    s.sample_into(i, out.data_ptr())
                s.sync()
                best = min(best, time.perf_counter() - t)
            took.append(best / 20)
        print(f"4096 receivers {took[0] * 1e6:.1f} us, 16384 receivers {took[1] * 1e6:.1f} us", flush=True)
        assert took[1] < 3.2 * took[0]
    finally:
        s.close()
