"""Which random word rounds which population of an F16 step: word i of the cell's
sequence rounds plane i, so a checkpoint continues on the same bits however the kernel
orders its planes.

One step is taken from the same populations in FP64 and in F16.  The FP64 values,
rounded with the words worked out here from the definition, are the F16 values, but
where FP32 arithmetic lands on the other side of a threshold.  An FP32 error of e in a
scaled value flips 2 e / spacing of them: e is about 3e-7 (2.3e-7 mean, per unit weight)
and the spacing at least 2^-18 for |value| >= 2^-8, so some 0.06 to 0.15 at the smallest
values and half that for each doubling.  Another word agrees on f^2 + (1 - f)^2 of
them for values at the fraction f of the spacing, 2/3 on average over f.  The line
between, for every plane: 0.8."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def words(ncell, step, q):
    """(q, ncell) words: the key of (cell, step), then the congruential sequence."""
    with np.errstate(over="ignore"):
        h = np.arange(ncell, dtype=np.uint32) * np.uint32(0x9E3779B1)
        h = h + np.uint32(step * 0x85EBCA77 & 0xFFFFFFFF)
        h ^= h >> np.uint32(16)
        h = h * np.uint32(0x85EBCA6B)
        h ^= h >> np.uint32(13)
        h = h * np.uint32(0xC2B2AE35)
        h ^= h >> np.uint32(16)
        out = np.empty((q, ncell), np.uint32)
        for i in range(q):
            out[i] = h
            h = h * np.uint32(0x4C957F2D) + np.uint32(0x2545F491)
    return out


@pytest.mark.parametrize("lattice,dims", [("D2Q37", (131, 97, 1)), ("D3Q39", (37, 22, 17))])
def test_plane_takes_its_word(lattice, dims):
    import torch

    from paper_2302_04741_amd import _lib, sim, workloads

    w = _lib.lattice_table(lattice)[1]
    q, n = len(w), int(np.prod(dims))
    scale = 2.0 ** np.round(-np.log2(w))[:, None]
    wl = workloads.random_smooth(lattice, dims, seed=5, tau_hat=0.75)

    half = sim.from_workload(wl, storage="f16dev")
    half.step(3)
    before = half.get_populations().view(torch.float16).cpu().numpy().astype(np.float64)
    half.step(1)
    got = half.get_populations().view(torch.float16).cpu().numpy().reshape(q, n)

    full = sim.from_workload(wl, storage="f64")
    full.set_populations(torch.from_numpy(before.reshape(q, n) / scale).cuda())
    full.step(1)
    v = full.get_populations().view(torch.float64).cpu().numpy().reshape(q, n) * scale
    half.close()
    full.close()

    bits = v.astype(np.float32).view(np.uint32)
    mag = bits & np.uint32(0x7FFFFFFF)
    up = (mag + (words(n, 3, q) >> np.uint32(19))) & np.uint32(0xFFFFE000)
    want = (up | (bits & np.uint32(0x80000000))).view(np.float32).astype(np.float16)
    large = np.abs(v) >= 2.0 ** -8
    for i in range(q):
        m = large[i]
        assert m.sum() > 200
        same = float((got[i][m] == want[i][m]).mean())
        assert same > 0.8, (i, same)
