"""The split-screen network's kernels at row counts where the tiles of 32 rows,
the wavefronts of a workgroup and the workgroups of a launch run out: forward
scores and the gradient against the reference, with the bounds of the
screen's own tests (bfloat16 roundings that fall the other way)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import screen as S  # noqa: E402
from paper_2509_01827_amd import mct2d  # noqa: E402

pytestmark = pytest.mark.gpu

TILE = 32


def _data(n, seed):
    rng = np.random.default_rng(seed)
    p = rng.normal(0.0, 0.3, S.N_PARAMS).astype(np.float32)
    X = rng.normal(0.0, 1.0, (n, S.N_IN)).astype(np.float32)
    y = (rng.random(n) < 0.2).astype(np.float32)
    return p, X, y


def _forward(m, X):
    out = torch.full((len(X) + 3,), -7.0, dtype=torch.float32, device="cuda")
    m.forward(torch.from_numpy(X).cuda(), out[:len(X)])
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.all(got[len(X):] == -7.0)
    return got[:len(X)]


# one row; around a tile; around one tile per workgroup of the forward (1024);
# the second tile of a wavefront.  A row's score does not depend on the others,
# so many rows give bit for bit what slices of a few give, and those are
# compared with the reference.
@pytest.mark.parametrize("n", [1, 31, 32, 33, 1024 * TILE, 1024 * TILE + 1, 4 * 1024 * TILE + 5])
def test_forward_rows(n):
    p, X, _ = _data(n, 21)
    m = mct2d.Mlp()
    m.set_params(p)
    got = _forward(m, X)
    if n <= 33:
        want = S.forward(p.astype(np.float64), X.astype(np.float64), emulate_bf16=True)
        assert np.all(np.abs(got - want) <= 2e-3 * (1.0 + np.abs(want)))
    for r in list(range(0, n, 9973)) + [max(0, n - 50)]:
        assert np.array_equal(got[r:r + 50], _forward(m, X[r:r + 50])), r


# one row; one tile and two; every workgroup one wavefront, one more; every
# wavefront one tile, and the second tile of some
@pytest.mark.parametrize("n", [1, 32, 33, 256 * TILE, 256 * TILE + 1, 512 * TILE + 1, 2048 * TILE, 2048 * TILE + 33])
def test_gradient_rows(n):
    p, X, y = _data(n, 22)
    m = mct2d.Mlp()
    m.set_params(p)
    xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    loss, g = m.gradient(xd, yd, pos_weight=3.0)
    again, g2 = m.gradient(xd, yd, pos_weight=3.0)
    assert loss == again and np.array_equal(g, g2)  # the sums have one order
    wl, wg = S.loss_and_grad(p.astype(np.float64), X.astype(np.float64), y.astype(np.float64), 3.0, True)
    assert loss == pytest.approx(wl, rel=1e-5)
    for a, b in ((0, 640), (640, 704), (704, 4800), (4800, 4864), (4864, 4928), (4928, 4929)):
        err = np.linalg.norm(g[a:b] - wg[a:b]) / max(np.linalg.norm(wg[a:b]), 1e-30)
        assert err < 5e-3, (n, a, err)
