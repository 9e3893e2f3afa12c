"""Export and import of the populations (dense rows <-> padded rows): bit for bit, at
any alignment of the dense side, against the runtime's own 2-D copy (taken for
addresses not aligned to the stored type and for small states), at row lengths around
the 16-byte chunks and the 64-value padding; the states are just large enough for the
row kernel (6 MiB), a few smaller."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZE = {"f64": 8, "f32": 4, "f16dev": 2}


def _sim(lattice, dims, storage):
    from paper_2302_04741_amd import sim

    return sim.Sim(lattice, dims, 0.8, 1.0, 0.0, 1.0, storage=storage)


def _call(name, s, buf, off):
    from paper_2302_04741_amd import _lib

    _lib.check(getattr(_lib.load(), name)(s.handle, ctypes.c_void_p(buf.data_ptr() + off)))


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
@pytest.mark.parametrize("lattice,dims", [
    ("D2Q37", (1, 60000)), ("D2Q37", (2, 45000)), ("D2Q37", (3, 30000)), ("D2Q37", (5, 19000)),
    ("D2Q37", (7, 13000)), ("D2Q37", (9, 11000)), ("D2Q37", (16, 6000)), ("D2Q37", (63, 1500)),
    ("D2Q37", (65, 1500)), ("D2Q37", (127, 800)), ("D2Q37", (1017, 100)), ("D2Q37", (1025, 90)),
    ("D2Q37", (4099, 23)), ("D2Q37", (9001, 11)), ("D2Q37", (90001, 1)),
    ("D3Q39", (5, 30, 600)), ("D3Q39", (129, 20, 40)),
    ("D2Q37", (3, 5)), ("D2Q37", (65, 3)), ("D3Q39", (5, 3, 2)),
])
def test_rows_bit_for_bit(lattice, dims, storage):
    import torch

    s = _sim(lattice, dims, storage)
    n = s.population_bytes()
    rng = np.random.default_rng(n)
    src = torch.from_numpy(np.frombuffer(rng.bytes(n + 64), np.uint8).copy()).cuda()
    offsets = [0, SIZE[storage], 3 * SIZE[storage], 16 - SIZE[storage]]
    for into in offsets + [1]:  # an odd address goes through the runtime's copy
        want = src[into:into + n].clone()
        _call("lbm_set_populations", s, src, into)
        for out in offsets + [1]:
            dst = torch.full((n + 64,), 0xA5, dtype=torch.uint8, device="cuda")
            _call("lbm_get_populations", s, dst, out)
            assert torch.equal(dst[out:out + n], want), (into, out)
            assert bool((dst[:out] == 0xA5).all()) and bool((dst[out + n:] == 0xA5).all())
    s.close()
