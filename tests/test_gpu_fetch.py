"""Query results through the pinned buffers: fields and split codes of models
whose arrays end before, at and behind the buffers' size (1 MB each), and of
batch specimens whose arrays start at any byte, against the same state read
another way."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2509_01827_amd import mct2d, workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


# (nodes: 9; one control block short of a buffer; exactly one, two; ragged beyond)
@pytest.mark.parametrize("nx,ny", [(2, 2), (250, 260), (255, 255), (511, 255), (521, 263), (700, 401)])
def test_grid_fields_equal_the_bound_arrays(nx, ny):
    cfg = W.plate(nx, ny, 1.0e-4 * nx, 1.0e-4 * ny, traction=2.0e7, jitter=0.02, seed=W.BASE_SEED + nx,
                  notch_len=nx // 2, name="fetch")
    m = mct2d.Model()
    mct2d._setup(m, cfg)
    nn = (nx + 1) * (ny + 1)
    bufs = [torch.zeros(nn, dtype=torch.float64, device="cuda") for _ in range(6)]
    m.bind_device_buffers(*bufs)
    m.finalize()
    for n in (25, 2):
        m.step(n)
        u, v, codes = m.field(mct2d.FIELD_U), m.field(mct2d.FIELD_V), m.split_codes()
        torch.cuda.synchronize()
        b = [x.cpu().numpy() for x in bufs]
        k = m.info()["step"] & 1  # (ux of even and odd steps, uy alike, vx, vy)
        assert np.array_equal(u[0], b[k]) and np.array_equal(u[1], b[2 + k])
        assert np.array_equal(v[0], b[4]) and np.array_equal(v[1], b[5])
        want = np.zeros(nx * ny, np.uint8)
        el, en, ex = cfg["notch"]
        want[np.asarray(el, int)] = 0x80 | (np.asarray(en) << 2) | np.asarray(ex)
        lg = m.crack_set()
        want[lg["elem"]] = 0x80 | (lg["entry"] << 2) | lg["exit"]
        assert np.array_equal(codes, want)
    if nx > 2:
        assert np.abs(u[1]).max() > 0 and np.abs(v[1]).max() > 0


@pytest.mark.parametrize("kind,nx,ny", [("tri", 3, 2), ("tri", 255, 255), ("tri", 300, 250), ("quad", 110, 100)])
def test_mesh_fields_equal_the_checkpoint(kind, nx, ny):
    make = W.tri_plate if kind == "tri" else W.quad_plate
    cfg = make(nx, ny, 1.0e-4 * nx, 1.0e-4 * ny, traction=2.0e7, notch_len=0.5e-4 * nx)
    m = mct2d.from_config(cfg)
    m.step(31)
    nn, ne = len(cfg["X"]), len(cfg["conn"])
    raw = np.frombuffer(m.checkpoint(), np.uint8)
    f = np.frombuffer(raw[64:64 + 32 * nn].tobytes(), np.float64).reshape(2, nn, 2)  # u, v behind 64 bytes
    for which, want in ((mct2d.FIELD_U, f[0]), (mct2d.FIELD_V, f[1])):
        x, y = m.field(which)
        assert np.array_equal(x, want[:, 0]) and np.array_equal(y, want[:, 1])
    assert np.array_equal(m.split_codes(), raw[64 + 32 * nn:64 + 32 * nn + ne])
    assert np.abs(f).max() > 0


def test_batch_specimens_at_any_offset():
    cfgs = W.batch_specimens(7, seed=W.BASE_SEED + 9, nx_range=(9, 41), ny_range=(7, 33))
    b = mct2d.batch_from_configs(cfgs)
    b.step(300)
    for s, c in enumerate(cfgs):
        one = mct2d.from_config(c, tile=1)
        one.step(300)
        b.select(s)
        assert np.array_equal(b.split_codes(), one.split_codes())
        for which in (mct2d.FIELD_U, mct2d.FIELD_V):
            assert all(np.array_equal(p, q) for p, q in zip(b.field(which), one.field(which)))
