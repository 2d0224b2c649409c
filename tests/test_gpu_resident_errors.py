"""A launch of the resident step that gave up (its error word set from the
host) is reported by mct_sync, mct_checkpoint and every query that waits for
the device, whatever launch choice is made afterwards, until the state is
restored."""
import pytest

torch = pytest.importorskip("torch")

from shimmed import run  # noqa: E402

pytestmark = pytest.mark.gpu

CODE = """
cfgs = CONFIGS()
for name, cfg in cfgs.items():
    mesh = cfg.get("conn") is not None
    word("shim_watch_bytes", 8 if mesh else 16, ctypes.c_size_t)  # finalize clears the error word
    m = mct2d.from_config(cfg)
    err = word("shim_cleared", type=ctypes.c_void_p)
    m.step(120)
    saved, before = m.checkpoint(), state(m)
    m.step(20)
    m.sync()
    assert shim.shim_poke(ctypes.c_void_p(err), 1) == 0
    calls = dict(sync=m.sync, info=m.info, u=lambda: m.field(mct2d.FIELD_U), v=lambda: m.field(mct2d.FIELD_V),
                 a=lambda: m.field(mct2d.FIELD_A), sigma=lambda: m.field(mct2d.FIELD_SIGMA_EDGE), codes=m.split_codes,
                 cracks=m.crack_set, tips=m.tips, energies=m.energies, checkpoint=m.checkpoint)
    for tile in (0, 1):
        m.set_launch(tile, True)
        for call, f in calls.items():
            try:
                f()
            except mct2d.MctError as e:
                assert "did not answer" in str(e), (name, tile, call, str(e))
            else:
                raise AssertionError((name, tile, call, "no error"))
    m.restore(saved)
    m.sync()
    assert all(np.array_equal(a, b) for a, b in zip(state(m), before))
    m.close()
    print(name, "ok", flush=True)
b = mct2d.batch_from_configs(W.batch_specimens(3, seed=W.BASE_SEED + 9, nx_range=(9, 20), ny_range=(7, 16)))
b.step(30)
b.sync()
b.split_codes()
b.checkpoint()
"""


def test_a_launch_that_gave_up_is_reported(tmp_path):
    run(CODE, tmp_path)
