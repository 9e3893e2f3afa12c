"""Host side of the Python binding, on the CPU: the layouts of input arrays it takes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

RECORD = np.zeros(6, dtype=[("a", "f8"), ("b", "i2")])
RECORD["a"] = np.arange(6.0)
CASES = {
    "plain": (np.arange(6.0).reshape(2, 3), (2, 3)),
    "scalar": (1.5, (4,)),
    "broadcast row": (np.arange(3.0), (2, 3)),
    "list": ([1.0, 2.0], (2,)),
    "float32": (np.arange(4, dtype=np.float32), (4,)),
    "big endian": (np.arange(4, dtype=">f8"), (4,)),
    "fortran order": (np.asfortranarray(np.arange(6.0).reshape(2, 3)), (2, 3)),
    "read only": (np.broadcast_to(np.float64(2.0), (3,)), (3,)),
    "reversed": (np.arange(4.0)[::-1], (4,)),
    "every other": (np.arange(8.0)[::2], (4,)),
    "one value reversed": (np.array([3.0])[::-1], (1,)),
    "one column reversed": (np.array([[1.0], [2.0]])[:, ::-1], (2, 1)),
    "one row reversed": (np.arange(3.0).reshape(1, 3)[::-1], (1, 3)),
    "one value of a packed record": (RECORD["a"][4:5], (1,)),
    "a packed record": (RECORD["a"], (6,)),
    "unaligned": (np.frombuffer(bytearray(3) + bytearray(np.arange(4.0).tobytes()), np.float64,
                                offset=3), (4,)),
    "no values": (np.zeros((2, 0)), (2, 0)),
    "tensor": (torch.arange(6.0).reshape(3, 2).t(), (2, 3)),
}


@pytest.mark.parametrize("name", CASES)
def test_input_layouts(name, monkeypatch):
    from paper_2302_04741_amd import sim

    monkeypatch.setattr(torch.Tensor, "record_stream", lambda self, stream: None)
    a, shape = CASES[name]
    keep = []
    t = sim._as_device(torch, a, shape, torch.device("cpu"), None, keep)
    assert t.dtype == torch.float64 and tuple(t.shape) == shape and t.is_contiguous()
    assert np.array_equal(t.numpy(), np.broadcast_to(np.asarray(a, dtype=np.float64), shape))
