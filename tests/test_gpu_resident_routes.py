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
    word("shim_no_launch", 1)  # (the route only)
    m.step(40)
    assert word("shim_cooperative") == int(resident), (nx, ny, kw)
    m.close()
"""

STEPS = """
# fewest steps: 6 on fewer than 32 tiles (15 x 15 nodes each), 4 on more; 10 on meshes
tri = W.tri_plate(40, 16, 0.1, 0.04, notch_len=0.05, traction=8.0e6)
for cfg, least in (((20, 16), 6), ((74, 89), 6), ((75, 89), 4), (tri, 10)):
    if isinstance(cfg, tuple):
        cfg = W.plate(*cfg, 1.0e-4 * cfg[0], 1.0e-4 * cfg[1], traction=2.0e7, notch_len=cfg[0] // 2, name="route")
    m, ref = mct2d.from_config(cfg), mct2d.from_config(cfg, tile=1)
    word("shim_cooperative", 0)
    m.step(least - 1)
    m.sync()
    assert word("shim_cooperative") == 0, least
    m.step(least)
    m.sync()
    assert word("shim_cooperative") == 1, least
    ref.step(2 * least - 1)
    assert all(np.array_equal(a, b) for a, b in zip(state(m), state(ref)))
"""


@pytest.mark.parametrize("code", [SIZES, STEPS], ids=["sizes", "steps"])
def test_routes(code, tmp_path):
    run(code, tmp_path)


def test_the_route_is_reported(tmp_path):
    """mct_get_resident: the fewest steps as above, 0 with a tile shape, without graphs, for a batch, screened."""
    run("""
plate = W.plate(75, 89, 0.0075, 0.0089, notch_len=30, name="route")
for cfg, least in ((W.small_cases()["plate40x40"], 6), (plate, 4), (W.tri_plate(40, 16, 0.1, 0.04), 10)):
    m = mct2d.from_config(cfg)
    assert m.resident() == least
    m.set_launch(1, True)
    assert m.resident() == 0
    m.set_launch(0, False)
    assert m.resident() == 0
    m.set_launch(0, True)
    assert m.resident() == least
m = mct2d.from_config(plate)
mlp = mct2d.Mlp()
mlp.set_params(np.zeros(mct2d.N_PARAMS, np.float32))
m.screen_enable(mlp, 0.0, 50)
assert m.resident() == 0
assert mct2d.batch_from_configs([plate, plate]).resident() == 0
""", tmp_path)
