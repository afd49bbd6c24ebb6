"""State transfers: what is written is read back, element by element.

A chunk holds up to 256 K values: the cases are a small part of a chunk, most of
one, and several chunks whose last is short, so that one and several host
threads and both buffers of a thread take part. FP64 handles return the
very values, 32-bit handles the nearest FP32 ones; read_elements, which copies
single groups, has to agree.
"""
import numpy as np
import pytest

from paper_2107_06640_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,kernel", [("fp64", "plain"), ("fp32", "tuned")])
@pytest.mark.parametrize("order,cells", [(3, (3, 3, 3)), (7, (3, 4, 4)), (7, (6, 9, 7)), (4, (12, 13, 12))])
def test_write_then_read(precision, kernel, order, cells):
    from paper_2107_06640_amd import seis
    mesh = inputs.box_mesh(*cells, lengths=tuple(500.0 * n for n in cells))
    mats = inputs.uniform_materials(mesh, **inputs.ROCK)
    s = seis.from_mesh(mesh, mats, order, precision=precision, kernel=kernel)
    try:
        rng = np.random.default_rng(3)
        for _ in range(2):  # the second transfer reuses the staging
            q = rng.standard_normal((mesh.n_elements, s.B, 9))
            s.write(q)
            got, _ = s.read()
            want = q if precision == "fp64" else q.astype(np.float32).astype(np.float64)
            assert np.array_equal(got, want)
        ids = np.unique(rng.integers(0, mesh.n_elements, 40))
        assert np.array_equal(s.read_elements(ids), want[ids])
    finally:
        s.close()
