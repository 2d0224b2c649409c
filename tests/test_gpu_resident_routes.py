"""Which requests the resident step takes and which the per-step kernels: by
the size of the grid and the number of steps (where each is faster)."""
import pytest

torch = pytest.importorskip("torch")

from shimmed import run  # noqa: E402

pytestmark = pytest.mark.gpu

SIZES = """
# binary64: tiles of 768 ring elements (26 x 27 nodes each), at most 256; binary32: 31 x 31 nodes
for nx, ny, kw, resident in ((415, 431, {}, True), (416, 431, {}, False), (495, 495, {}, False),
                             (415, 431, dict(smoothing="subcell"), True), (415, 432, dict(smoothing="subcell"), False),
                             (495, 495, dict(precision=32), True), (496, 495, dict(precision=32), False)):
    cfg = W.plate(nx, ny, 1.0e-4 * nx, 1.0e-4 * ny, traction=2.0e7, notch_len=nx // 2, name="route")
    cfg.update(kw)
    m = mct2d.from_config(cfg)
    word("shim_cooperative", 0)
    m.step(40)
    m.sync()
    assert word("shim_cooperative") == int(resident), (nx, ny, kw)
    m.close()
"""


def test_grid_sizes(tmp_path):
    run(SIZES, tmp_path)
