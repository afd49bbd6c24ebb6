"""The BF16 predictor's product shape follows from the order, however the handle was set up.

16x16x16 and 16x16x32 products round differently, so a handle's results may not depend on
whether it was tuned: on a tuning cache, with tuning off, with a fixed tile, or where the largest
cluster is too small to tune on. Two row tiles a product where the basis has an even count of
16-row tiles (orders 4, 6 and 7).
"""
import pytest

from paper_2107_06640_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [3, 4, 5, 6, 7])
def test_shape_does_not_depend_on_tuning(order, tmp_path, monkeypatch):
    from paper_2107_06640_amd import seis
    mesh, mats = inputs.coupled_box(6, 6, 4, cell=500.0, water_layers=1, jitter=0.1, seed=7)
    monkeypatch.setenv("SEIS_TUNE_CACHE", str(tmp_path / "tune.txt"))
    shapes, source = {}, {}
    for how, tune, kw in (("measured", None, dict(mc_min=0)), ("cached", None, dict(mc_min=0)), ("off", "0", dict(mc_min=0)),
                          ("tile", None, dict(mc_min=0, tile=32)), ("small", None, {})):
        if tune is None:
            monkeypatch.delenv("SEIS_TUNE", raising=False)
        else:
            monkeypatch.setenv("SEIS_TUNE", tune)
        s = seis.from_mesh(mesh, mats, order, precision="bf16", **kw)
        try:
            shapes[how], source[how] = s.info()["shape"], s.info()["launch_source"]
        finally:
            s.close()
    assert source == {"measured": 1, "cached": 2, "off": 0, "tile": 0, "small": 0}
    assert set(shapes.values()) == {1 if order in (4, 6, 7) else 0}, shapes
