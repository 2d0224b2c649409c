"""Scores of the split-screen network at the row counts where its launch
changes: 512 workgroups of four wavefronts take tiles of 32 rows, first every
workgroup's first wavefront (up to 512 tiles), last the second tile of a
wavefront (from 2 049 on).  Every row is compared: bit for bit with launches
of few rows (a row's score does not depend on the others), and with the
reference within a rounding of the hidden layers that falls the other way (a
bfloat16 step, 2^-8, of a value up to 8 under a weight up to 1.2)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import screen as S  # noqa: E402
from paper_2509_01827_amd import mct2d  # noqa: E402

pytestmark = pytest.mark.gpu

TILE = 32


@pytest.mark.parametrize("n", [512 * TILE - 1, 512 * TILE, 512 * TILE + 1, 2048 * TILE, 2048 * TILE + 1])
def test_every_row(n):
    rng = np.random.default_rng(23)
    p = rng.normal(0.0, 0.3, S.N_PARAMS).astype(np.float32)
    X = rng.normal(0.0, 1.0, (n, S.N_IN)).astype(np.float32)
    m = mct2d.Mlp()
    m.set_params(p)

    def scores(x):
        out = torch.full((len(x) + 3,), -7.0, dtype=torch.float32, device="cuda")
        m.forward(torch.from_numpy(x).cuda(), out[:len(x)])
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert np.all(got[len(x):] == -7.0)
        return got[:len(x)]

    got = scores(X)
    parts = np.concatenate([scores(X[r:r + 1000]) for r in range(0, n, 1000)])
    assert np.array_equal(got, parts)
    want = S.forward(p.astype(np.float64), X.astype(np.float64), emulate_bf16=True)
    assert np.all(np.abs(got - want) <= 0.05 * (1.0 + np.abs(want)))
