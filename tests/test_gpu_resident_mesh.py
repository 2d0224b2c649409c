"""The resident step of an unstructured mesh (many steps per launch, the state
on the chip) against the oracle, bit for bit: triangles and quadrilaterals,
every loading, node numberings without locality, meshes of one patch, patches
whose candidate and boundary lists overflow; and against the per-step kernels
at the sizes where the patch classes change."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2509_01827_amd import mct2d, workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


def _shuffled(cfg, seed):
    nn = len(cfg["X"])
    pn = np.argsort(W.uniform01(seed, nn), kind="stable")
    inv = np.empty(nn, np.int64)
    inv[pn] = np.arange(nn)
    vn, vm, vv = cfg["vbc"]
    return dict(cfg, X=np.ascontiguousarray(cfg["X"][pn]), Y=np.ascontiguousarray(cfg["Y"][pn]),
                conn=np.ascontiguousarray(inv[np.asarray(cfg["conn"], np.int64)].astype(np.int32)),
                traction_nodes=np.ascontiguousarray(inv[np.asarray(cfg["traction_nodes"], np.int64)].astype(np.int32)),
                vbc=(np.ascontiguousarray(inv[np.asarray(vn, np.int64)].astype(np.int32)), vm, vv))


def _weak(cfg, mean):
    """Low, scattered toughness: many cracks, many free edges."""
    return dict(cfg, gc_uniform=0.0, gc_field=W.weibull_gc(W.BASE_SEED + 7, len(cfg["conn"]), 6.0, mean))


def _pulled(cfg):
    """Every node of the lower half held at a velocity of its own: more
    prescribed nodes than a patch keeps at hand."""
    X, Y = cfg["X"], cfg["Y"]
    n = np.flatnonzero(Y < 0.5 * Y.max()).astype(np.int32)
    v = np.stack([0.5 * X[n] / X.max(), -3.0 + Y[n] / Y.max()], 1)
    mask = np.where(n % 3 == 0, 3, np.where(n % 3 == 1, 1, 2)).astype(np.uint8)
    return dict(cfg, vbc=(n, mask, np.ascontiguousarray(v)), t_ramp=1.0e-6)


def _cases():
    tri = W.tri_plate(40, 16, 0.1, 0.04, notch_len=0.05, traction=8.0e6)
    quad = W.quad_plate(24, 10, 0.1, 0.04, notch_len=0.05, traction=8.0e6)
    grid = W.as_unstructured_q4(dict(W.small_cases()["plate70x37_jitter"]))
    return {
        "tri_one_patch": W.tri_plate(12, 10, 0.012, 0.01, notch_len=0.006, traction=8.0e6),
        "tri_plate": tri, "tri_shuffled": _shuffled(tri, W.BASE_SEED + 3), "tri_gamma": dict(tri, gamma=2.0),
        "tri_cylinder": W.tri_cylinder(h=5.0e-3), "tri_fragment": W.tri_fragment(36, 30, 1.0e-3),
        "tri_weak": _weak(W.tri_fragment(44, 32, 1.0e-3), 0.05), "tri_pulled": _pulled(tri),
        "quad_one_patch": W.quad_plate(5, 4, 0.005, 0.004, notch_len=0.002, traction=8.0e6),
        "quad_plate": quad, "quad_shuffled": _shuffled(quad, W.BASE_SEED + 4), "quad_grid": grid,
        "quad_weak": _weak(W.as_unstructured_q4(W.fragmentation(41, 33, 1.0e-3, seed=W.BASE_SEED + 5)), 0.05),
        "quad_curve": W.as_unstructured_q4(W.pulse_plate(48, 32, 0.048, 0.032, peak=2e6, steps=900, t0=2e-6,
                                                         tau=4e-6)),
        "quad_pulled": _pulled(quad),
    }


def _same(m, o, label):
    lg, ol, st = m.crack_set(), o.log(), o.state()
    for k in ("step", "elem", "entry", "exit", "G"):
        assert np.array_equal(lg[k], ol[k]), (label, k)
    assert np.array_equal(m.split_codes(), st["split"]), label
    (ux, uy), (vx, vy) = m.field(mct2d.FIELD_U), m.field(mct2d.FIELD_V)
    for a, b in ((ux, "ux"), (uy, "uy"), (vx, "vx"), (vy, "vy")):
        assert np.array_equal(a, st[b]), (label, b, np.abs(a - st[b]).max())
    assert m.info()["dissipated"] == o.info()["Ud"], label


@pytest.mark.parametrize("name", ["tri_one_patch", "tri_plate", "tri_shuffled", "tri_gamma", "tri_cylinder",
                                  "tri_fragment", "tri_weak", "tri_pulled", "quad_one_patch", "quad_plate",
                                  "quad_shuffled", "quad_grid", "quad_weak", "quad_curve", "quad_pulled"])
def test_small_meshes_against_the_oracle(name, oracle_mod):
    cfg = _cases()[name]
    m = mct2d.from_config(cfg)
    o = oracle_mod.Oracle(cfg)
    # requests of one launch, two launches, and per-step kernels between them
    for n in (1, 10, 99, 9, 2, 541, 300):
        m.step(n)
        o.step(n)
        _same(m, o, (name, n))
    ns = len(o.log()["elem"])
    print(name, "splits", ns, flush=True)
    assert ns > 0 or "one_patch" in name or "pulled" in name


def _fields(m):
    return m.field(mct2d.FIELD_U) + m.field(mct2d.FIELD_V) + (m.split_codes(),)


# 512-thread patches; the largest mesh that takes them and the next (190 x 256
# nodes); 768-thread patches near their limit; meshes too large for the chip
@pytest.mark.parametrize("kind,nx,ny", [("tri", 150, 99), ("tri", 255, 189), ("tri", 255, 190), ("tri", 435, 370),
                                        ("tri", 480, 400), ("quad", 80, 60), ("quad", 100, 80), ("quad", 101, 81),
                                        ("quad", 250, 105), ("quad", 290, 120)])
def test_patch_classes_against_the_step_kernels(kind, nx, ny):
    make = W.tri_plate if kind == "tri" else W.quad_plate
    cfg = make(nx, ny, 1.0e-4 * nx, 1.0e-4 * ny, traction=2.0e7, notch_len=0.5e-4 * nx, gc=0.3)
    a, b = mct2d.from_config(cfg), mct2d.from_config(cfg, tile=1)
    for n in (120, 33):
        a.step(n)
        b.step(n)
        assert all(np.array_equal(x, y) for x, y in zip(_fields(a), _fields(b)))
        la, lb = a.crack_set(), b.crack_set()
        assert all(np.array_equal(la[k], lb[k]) for k in la)
        assert a.info()["dissipated"] == b.info()["dissipated"]
    assert len(la["elem"]) > 0


def test_checkpoint_and_kernel_changes_between_launches():
    cfg = _cases()["tri_plate"]
    a, b = mct2d.from_config(cfg), mct2d.from_config(cfg)
    a.step(101)
    saved = a.checkpoint()
    a.step(300)
    b.step(5)
    b.restore(saved)
    b.step(64)
    b.set_launch(1, True)  # per-step kernels, then resident again
    b.step(33)
    b.set_launch(0, True)
    b.step(203)
    assert all(np.array_equal(x, y) for x, y in zip(_fields(a), _fields(b)))
    la, lb = a.crack_set(), b.crack_set()
    assert all(np.array_equal(la[k], lb[k]) for k in la)


def test_two_meshes_on_two_streams():
    cfgs = [_cases()["tri_weak"], _cases()["quad_plate"]]
    streams = [torch.cuda.Stream() for _ in cfgs]
    ms = [mct2d.from_config(c, stream=s.cuda_stream) for c, s in zip(cfgs, streams)]
    for _ in range(4):
        for m in ms:
            m.step(60)
    for m, c in zip(ms, cfgs):
        r = mct2d.from_config(c, tile=1)
        r.step(240)
        assert all(np.array_equal(x, y) for x, y in zip(_fields(m), _fields(r)))
