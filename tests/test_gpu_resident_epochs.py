"""The resident step's exchange words carry the step they are of in 21 bits:
models that take more steps than that, and buffers made anew at any count, go
on bit for bit as a model restored from a checkpoint shortly before."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2509_01827_amd import mct2d, workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu

TAGS = 1 << 21


def _model(kind):
    if kind == "tri":  # two patches
        return mct2d.from_config(W.tri_plate(20, 10, 0.02, 0.01, notch_len=0.01, traction=1.0e4))
    return mct2d.from_config(W.plate(20, 16, 0.02, 0.016, traction=1.0e4, notch_len=10, name="epochs"))


def _same(a, b):
    for which in (mct2d.FIELD_U, mct2d.FIELD_V):
        assert all(np.array_equal(x, y) for x, y in zip(a.field(which), b.field(which)))


@pytest.mark.parametrize("kind", ["tri", "grid"])
@pytest.mark.parametrize("anew", [False, True], ids=["through", "anew"])
def test_more_steps_than_tags(kind, anew):
    a, b = _model(kind), _model(kind)
    for n in (TAGS - 1 - (1 << 20), 1 << 20):
        a.step(n)
        a.sync()
    assert np.abs(a.field(mct2d.FIELD_U)[1]).max() > 0
    saved = a.checkpoint()
    if anew:  # new buffers with TAGS - 1 steps behind them
        a.set_launch(1, True)
        a.set_launch(0, True)
    b.restore(saved)
    for n in (37, 600):
        a.step(n)
        b.step(n)
        _same(a, b)
