"""Where the runtime refuses a resident launch, or the memory of its exchange,
the per-step kernels take the steps, with the same results; a new launch
choice plans the resident step again."""
import pytest

torch = pytest.importorskip("torch")

from paper_2509_01827_amd import mct2d  # noqa: E402
from shimmed import CONFIGS, run  # noqa: E402

pytestmark = pytest.mark.gpu

LAUNCHES = """
for name, cfg in CONFIGS().items():
    m, ref = mct2d.from_config(cfg), mct2d.from_config(cfg, tile=1)
    word("shim_cooperative", 0)
    m.step(40)
    assert word("shim_cooperative") == 1
    for nth, n in ((1, 70), (2, 600)):  # at once; in the middle of a request
        word("shim_cooperative", 0)
        word("shim_refuse_launch", nth)
        m.step(n)
        m.step(30)  # (per-step kernels)
        assert word("shim_cooperative") == nth, (name, nth)
        word("shim_refuse_launch", 0)
        m.set_launch(0, True)
        m.step(25)
        assert word("shim_cooperative") == nth + 1, (name, nth)
    ref.step(40 + 70 + 30 + 25 + 600 + 30 + 25)
    assert all(np.array_equal(a, b) for a, b in zip(state(m), state(ref))), name
    m.sync()
    print(name, "ok", flush=True)
"""

ALLOCATIONS = """
for name, cfg in CONFIGS().items():
    m, ref = mct2d.from_config(cfg, tile=1), mct2d.from_config(cfg, tile=1)
    ref.step(80)
    saved = m.checkpoint()
    word("shim_mallocs", 0)
    m.set_launch(0, True)
    made = word("shim_mallocs")
    # a grid's plan comes last (two allocations), a mesh's first (one)
    for nth in ((1,) if cfg.get("conn") is not None else (made - 1, made)):
        m.set_launch(1, True)
        m.restore(saved)
        word("shim_mallocs", 0)
        word("shim_cooperative", 0)
        word("shim_refuse_malloc", nth)
        m.set_launch(0, True)
        word("shim_refuse_malloc", 0)
        m.step(80)
        assert word("shim_cooperative") == 0, (name, nth)
        assert all(np.array_equal(a, b) for a, b in zip(state(m), state(ref))), (name, nth)
        m.set_launch(0, True)
        m.step(80)
        assert word("shim_cooperative") == 1, (name, nth)
    m.sync()
    print(name, made, "ok", flush=True)
"""

SECOND_PROCESS = """
word("shim_strict", 1)
for name, cfg in CONFIGS().items():
    m, ref = mct2d.from_config(cfg), mct2d.from_config(cfg, tile=1)
    for n in (40, 600):
        m.step(n)
        ref.step(n)
        m.sync()
        assert all(np.array_equal(a, b) for a, b in zip(state(m), state(ref))), (name, n)
    print(name, word("shim_cooperative"), "ok", flush=True)
"""


def test_a_second_process_on_the_device(tmp_path):
    """The runtime gives cooperative launches to one process at a time."""
    m = mct2d.from_config(CONFIGS()["grid"])
    m.step(100)
    m.sync()
    run(SECOND_PROCESS, tmp_path)
    m.step(100)
    m.sync()


@pytest.mark.parametrize("code", [LAUNCHES, ALLOCATIONS], ids=["launches", "allocations"])
def test_refused(code, tmp_path):
    run(code, tmp_path)
