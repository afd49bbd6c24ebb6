"""State transfers of many chunks: each pinned buffer of a thread is used again and again.

A chunk holds up to 256 K values, and at most eight threads take chunks in turn, each with two
buffers. From 3 x 8 chunks on some thread fills a buffer a second time, which it may do only
after the kernel of its earlier chunk has read it (or, reading, after copying that chunk out).
"""
import numpy as np
import pytest

from paper_2107_06640_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_every_buffer_is_used_again(precision):
    from paper_2107_06640_amd import seis
    mesh = inputs.box_mesh(12, 13, 12, lengths=(6000.0, 6500.0, 6000.0))
    mats = inputs.uniform_materials(mesh, **inputs.ROCK)
    s = seis.from_mesh(mesh, mats, 7, precision=precision, kernel="plain")
    try:
        per = 256 * 1024 // (9 * s.B)
        chunks = -(-mesh.n_elements // per)
        assert chunks > 4 * 8 and mesh.n_elements % per  # the last one is short
        rng = np.random.default_rng(3)
        for _ in range(3):
            q = rng.standard_normal((mesh.n_elements, s.B, 9))
            s.write(q)
            got, _ = s.read()
            assert np.array_equal(got, q if precision == "fp64" else q.astype(np.float32).astype(np.float64))
    finally:
        s.close()
