"""A context that takes one mesh after another keeps one set of pinned buffers
for its query results, and gives it back when it is closed."""
import pytest

torch = pytest.importorskip("torch")

from shimmed import run  # noqa: E402

pytestmark = pytest.mark.gpu

CODE = """
for name, cfg in CONFIGS().items():
    held = []
    before = word("shim_pinned")
    m = mct2d.from_config(cfg)
    for _ in range(3):
        m.step(20)
        state(m)
        held.append(word("shim_pinned") - before)
        mct2d._setup(m, cfg)  # the mesh anew
        m.finalize()
    m.close()
    assert held[0] > 0 and held == held[:1] * 3, (name, held)
    assert word("shim_pinned") == before, name
    print(name, held, flush=True)
"""


def test_pinned_buffers_have_one_owner(tmp_path):
    run(CODE, tmp_path)
