"""A model on a stream with a mask of compute units steps with kernels that
keep to the mask: no resident launch, the same results."""
import pytest

torch = pytest.importorskip("torch")

from shimmed import run  # noqa: E402

pytestmark = pytest.mark.gpu

CODE = """
create = shim.shim_masked_stream
create.restype = ctypes.c_void_p
for words, resident in (([0xffffffff] * 8, True), ([0xffffffff] * 4 + [0] * 4, False), ([0x0fffffff] + [0xffffffff] * 7, False)):
    stream = create(len(words), (ctypes.c_uint32 * len(words))(*words))
    assert stream
    for name, cfg in CONFIGS().items():
        m, ref = mct2d.from_config(cfg, stream=stream), mct2d.from_config(cfg, tile=1)
        word("shim_cooperative", 0)
        m.step(130)
        assert word("shim_cooperative") == int(resident), (name, words)
        ref.step(130)
        assert all(np.array_equal(a, b) for a, b in zip(state(m), state(ref))), (name, words)
        m.close()
    print(words, "ok", flush=True)
"""


def test_masked_streams(tmp_path):
    run(CODE, tmp_path)
