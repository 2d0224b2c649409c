"""The resident step of an unstructured mesh in patches whose list of elements
with candidates fills up during a launch, against the oracle, bit for bit: the
step in which the list passes its capacity, the steps whose remaining
candidates are evaluated where the element is, and lists started again after
that.  Pre-split elements strewn over one patch of weak elements nearly
fill its list."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2509_01827_amd import mct2d, workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu

LAUNCH = 512  # steps per launch, at most


def _patches(cfg, parts):
    """Patch of every node: the recursive bisection of the coordinates into equal counts."""
    X, Y = np.asarray(cfg["X"]), np.asarray(cfg["Y"])
    part = np.empty(len(X), int)
    count = [0]

    def cut(ids, n):
        if n == 1:
            part[ids] = count[0]
            count[0] += 1
            return
        k, l = (X, Y) if np.ptp(X[ids]) >= np.ptp(Y[ids]) else (Y, X)
        ids = ids[np.lexsort((ids, l[ids], k[ids]))]
        at = len(ids) * (n // 2) // n
        cut(ids[:at], n // 2)
        cut(ids[at:], n - n // 2)

    cut(np.arange(len(X)), parts)
    return part


def _neighbours(T):
    """Element across each local edge, -1 outside the mesh."""
    nv = T.shape[1]
    a, b = T, np.roll(T, -1, 1)
    key = (np.minimum(a, b).astype(np.int64) * (T.max() + 1) + np.maximum(a, b)).ravel()
    order = np.argsort(key, kind="stable")
    nb = np.full(len(key), -1)
    same = np.flatnonzero(key[order][1:] == key[order][:-1])
    nb[order[same]], nb[order[same + 1]] = order[same + 1] // nv, order[same] // nv
    return nb.reshape(T.shape)


def _listed(nb, split, mine):
    """Elements of the patch that are intact and have a free edge."""
    return mine & ~split & ((nb < 0) | split[nb]).any(1)


def _crowded(cfg, threads):
    """The mesh with the list of a patch on its loaded edge nearly full, and that patch's elements."""
    T = np.asarray(cfg["conn"], int)
    nn, ne = len(cfg["X"]), len(T)
    room, per = (192, 160) if threads == 512 else (96, 0)
    parts = -(-nn // per) if per else 256
    part, nb = _patches(cfg, parts), _neighbours(T)
    X, Y = np.asarray(cfg["X"]), np.asarray(cfg["Y"])
    mid = np.argmin((X - 0.5 * X.max()) ** 2 + Y ** 2)
    mine = part[T[:, 0]] == part[mid]
    split = np.zeros(ne, bool)
    for e in np.flatnonzero(mine)[np.argsort(W.uniform01(W.BASE_SEED + 11, int(mine.sum())))]:
        if split.sum() == mine.sum() // 6:
            break
        if (nb[e] < 0).any() or split[nb[e]].any():
            continue
        split[e] = True
        if _listed(nb, split, mine).sum() > room:
            split[e] = False
    el = np.flatnonzero(split).astype(np.int32)
    notch = (el, np.zeros(len(el), np.uint8), np.ones(len(el), np.uint8))
    gc = np.where(mine, 1.0e-4, 1.0e6)
    return dict(cfg, notch=notch, gc_uniform=0.0, gc_field=gc), nb, split, mine, room


def _crossings(log, nb, split, mine, room, steps):
    """Steps after which the list is first longer than it may be, or again after a start over (launch by launch)."""
    split, at, where = split.copy(), 0, []
    for first in range(0, steps, LAUNCH):
        listed = _listed(nb, split, mine)
        n = int(listed.sum())
        while at < len(log["step"]) and log["step"][at] < min(first + LAUNCH, steps):
            if n > room:  # started over
                listed = _listed(nb, split, mine)
                n = int(listed.sum())
            split[log["elem"][at]] = True
            new = _listed(nb, split, mine) & ~listed
            listed |= new
            if n <= room < n + int(new.sum()):
                where.append(int(log["step"][at]) + 1)
            n += int(new.sum())
            at += 1
    return where


@pytest.mark.parametrize("kind,nx,ny,threads", [("tri", 39, 15, 512), ("tri", 230, 225, 768), ("quad", 110, 76, 768)])
def test_lists_that_fill_up(kind, nx, ny, threads, oracle_mod):
    make = W.tri_plate if kind == "tri" else W.quad_plate
    cfg, nb, split, mine, room = _crowded(make(nx, ny, 1.0e-3 * nx, 1.0e-3 * ny, traction=2.0e7), threads)
    m, o = mct2d.from_config(cfg), oracle_mod.Oracle(cfg)
    for n in (300, 150):
        m.step(n)
        o.step(n)
        lg, ol, st = m.crack_set(), o.log(), o.state()
        for k in ("step", "elem", "entry", "exit", "G"):
            assert np.array_equal(lg[k], ol[k]), (n, k)
        assert np.array_equal(m.split_codes(), st["split"])
        (ux, uy), (vx, vy) = m.field(mct2d.FIELD_U), m.field(mct2d.FIELD_V)
        for a, b in ((ux, "ux"), (uy, "uy"), (vx, "vx"), (vy, "vy")):
            assert np.array_equal(a, st[b]), (n, b)
        assert m.info()["dissipated"] == o.info()["Ud"]
        where = _crossings(ol, nb, split, mine, room, 300) if n == 300 else where
    print(kind, threads, "crossings", where, "splits", len(ol["step"]), flush=True)
    assert where  # the list passed its capacity within a launch
