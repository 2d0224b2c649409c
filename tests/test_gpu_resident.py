"""The resident step of a structured grid (many steps per launch, the state on
the chip) against the oracle, bit for bit, at the sizes where its tiles can go
wrong: grids of one tile, last tiles one node wide, and the smallest and
largest grids of each tile class.  The per-step kernels are compared on the
same grids (a chosen tile shape runs them)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2509_01827_amd import mct2d, workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


def _plate(nx, ny, **kw):
    # a strong traction on a notched plate with varying toughness: cracks run
    # within the first steps, through tile borders
    c = W.plate(nx, ny, 1.0e-4 * nx, 1.0e-4 * ny, traction=2.0e7, jitter=0.02, seed=W.BASE_SEED + nx,
                notch_len=max(1, nx // 2), gc=0.0, gc_field=W.weibull_gc(W.BASE_SEED + ny, nx * ny, 6.0, 1.0),
                name="resident%dx%d" % (nx, ny))
    c.update(kw)
    return c


def _state(m):
    return m.field(mct2d.FIELD_U) + m.field(mct2d.FIELD_V) + (m.split_codes(),)


CASES = [
    # one tile; last tiles one node wide (15 k + 1 nodes); several tiles
    (2, 2, {}), (14, 14, {}), (15, 15, {}), (30, 29, {}), (45, 16, {}), (63, 47, {}),
    (45, 31, dict(smoothing="subcell")), (45, 31, dict(precision=32)), (31, 45, dict(precision=32, smoothing="subcell")),
    (40, 33, dict(gamma=2.0)), (33, 40, dict(load_curve=W.pressure_pulse(t0=2.0e-7, tau=1.0e-6, t_end=1.0e-5))),
]


@pytest.mark.parametrize("nx,ny,kw", CASES, ids=lambda v: str(v) if isinstance(v, int) else "-".join(v) or "plain")
def test_small_grids_against_the_oracle(nx, ny, kw, oracle_mod):
    cfg = _plate(nx, ny, **kw)
    m = mct2d.from_config(cfg)
    o = oracle_mod.Oracle(cfg)
    # requests of one launch, two launches, and per-step kernels between them
    for n in (1, 4, 37, 3, 2, 541, 64):
        m.step(n)
        o.step(n)
        lg, ol, st = m.crack_set(), o.log(), o.state()
        for key in ("step", "elem", "entry", "exit", "G"):
            assert np.array_equal(lg[key], ol[key]), (n, key)
        ux, uy, vx, vy, codes = _state(m)
        assert np.array_equal(ux, st["ux"]) and np.array_equal(uy, st["uy"])
        assert np.array_equal(vx, st["vx"]) and np.array_equal(vy, st["vy"])
        assert np.array_equal(codes, st["split"])
        assert m.info()["dissipated"] == o.info()["Ud"]
    if nx > 2:
        assert len(ol["elem"]) > 0


def test_velocity_ramp_and_weibull(oracle_mod):
    cfg = W.fragmentation(47, 31, 1.0e-3, v=5.0, seed=W.BASE_SEED + 5)
    cfg["t_ramp"] = 1.0e-5
    m = mct2d.from_config(cfg)
    o = oracle_mod.Oracle(cfg)
    m.step(700)
    o.step(700)
    st = o.state()
    ux, uy, vx, vy, codes = _state(m)
    assert len(o.log()["elem"]) > 0
    assert np.array_equal(ux, st["ux"]) and np.array_equal(uy, st["uy"]) and np.array_equal(codes, st["split"])
    assert np.array_equal(vx, st["vx"]) and np.array_equal(vy, st["vy"])


# the largest grid of a tile class and the smallest of the next one, in each
# precision and smoothing; the last is too large for the chip
@pytest.mark.parametrize("nx,ny,kw", [
    (239, 239, {}), (240, 239, {}), (335, 351, {}), (336, 351, {}), (415, 431, {}), (416, 431, {}), (495, 495, {}),
    (496, 495, {}), (336, 352, dict(smoothing="subcell")), (416, 432, dict(precision=32)),
    (900, 100, dict(smoothing="subcell")), (100, 1500, dict(precision=32, smoothing="subcell"))],
    ids=lambda v: str(v) if isinstance(v, int) else "-".join(v) or "plain")
def test_tile_classes_against_the_step_kernels(nx, ny, kw):
    cfg = _plate(nx, ny, **kw)
    a, b = mct2d.from_config(cfg), mct2d.from_config(cfg, tile=1)
    for n in (120, 33):
        a.step(n)
        b.step(n)
        assert all(np.array_equal(x, y) for x, y in zip(_state(a), _state(b)))
        la, lb = a.crack_set(), b.crack_set()
        assert all(np.array_equal(la[k], lb[k]) for k in la)
        assert a.info()["dissipated"] == b.info()["dissipated"]
    assert len(la["elem"]) > 0


def test_checkpoint_between_launches():
    cfg = _plate(63, 47)
    a, b = mct2d.from_config(cfg), mct2d.from_config(cfg)
    a.step(101)
    saved = a.checkpoint()
    a.step(200)
    b.step(5)
    b.restore(saved)
    b.step(200)
    assert all(np.array_equal(x, y) for x, y in zip(_state(a), _state(b)))
    la, lb = a.crack_set(), b.crack_set()
    assert all(np.array_equal(la[k], lb[k]) for k in la)


def test_bound_buffers_hold_both_steps():
    """Caller-owned arrays are left as the per-step kernels leave them: u of
    the last step in the buffer of its parity, of the step before in the other."""
    cfg = _plate(45, 31)
    got = []
    for tile in (0, 1):
        m = mct2d.Model()
        mct2d._setup(m, cfg)
        nn = 46 * 32
        bufs = [torch.zeros(nn, dtype=torch.float64, device="cuda") for _ in range(6)]
        m.bind_device_buffers(*bufs)
        m.set_launch(tile, True)
        m.finalize()
        m.step(51)
        m.sync()
        got.append([b.cpu().numpy() for b in bufs])
        m.close()
    assert all(np.array_equal(x, y) for x, y in zip(*got))


def test_two_models_on_two_streams():
    """Two resident models stepped in turn on streams of their own."""
    cfgs = [_plate(63, 47), _plate(200, 120)]
    streams = [torch.cuda.Stream() for _ in cfgs]
    ms = [mct2d.from_config(c, stream=s.cuda_stream) for c, s in zip(cfgs, streams)]
    for _ in range(4):
        for m in ms:
            m.step(60)
    for m, c in zip(ms, cfgs):
        r = mct2d.from_config(c, tile=1)
        r.step(240)
        assert all(np.array_equal(x, y) for x, y in zip(_state(m), _state(r)))
