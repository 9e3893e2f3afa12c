"""Cache policies, sweep directions and launch shapes of the step, chosen by the size
of the populations: a periodic grid made of copies of a small one must evolve into
copies of what the small one evolves into (the small one is of the size every other
parity test runs at).

Tolerance: the kernels differ in access policy only, but each is compiled by itself
and may contract differently, a few units in the last place of the largest stored
value a step: 8 eps max|h| a step.  F16 (random bits keyed by the cell, so copies
differ) is held to FP32 at the storage's own bar for a few steps (2e-4, 2e-3 on u)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = {"f64": 2.0 ** -53, "f32": 2.0 ** -24}
STEPS = 5

# small grid, copies along each axis, and what the large one's size selects
TILED = [
    ("D2Q37", "f32", (100, 90), (8, 9), "both buffers cached, ragged rows"),
    ("D3Q39", "f64", (32, 16, 16), (2, 4, 4), "both buffers cached"),
    ("D2Q37", "f64", (96, 64), (8, 12), "end of the sweep kept"),
    ("D2Q37", "f64", (128, 128), (8, 8), "end of the sweep kept"),
    ("D2Q37", "f64", (192, 128), (8, 8), "end of the sweep kept"),
    ("D2Q37", "f32", (128, 128), (8, 8), "end of the sweep kept"),
    ("D2Q37", "f32", (181, 100), (8, 14), "end of the sweep kept, ragged rows"),
    ("D2Q37", "f32", (250, 100), (8, 20), "end of the sweep kept, 8 wavefronts a CU, ragged rows"),
    ("D3Q39", "f32", (48, 32, 24), (2, 3, 4), "end of the sweep kept"),
    ("D3Q39", "f32", (40, 40, 40), (4, 4, 4), "end of the sweep kept, 8 wavefronts a CU"),
    ("D3Q39", "f64", (45, 20, 20), (2, 4, 4), "end of the sweep kept, ragged rows"),
    ("D3Q39", "f64", (33, 30, 30), (4, 4, 4), "non-temporal loads throughout, ragged rows"),
]


def _fields(lattice, dims, seed):
    from paper_2302_04741_amd import workloads

    return workloads.random_smooth(lattice, dims, seed=seed, tau_hat=0.7, force_kind="uniform")


def _tile(a, dims, copies):
    nx, ny, nz = dims
    cx, cy, cz = copies
    lead = a.shape[:-1]
    a = a.reshape(lead + (nz, ny, nx))
    return np.ascontiguousarray(np.tile(a, (1,) * len(lead) + (cz, cy, cx))).reshape(lead + (-1,))


@pytest.mark.parametrize("lattice,storage,small,copies,what", TILED,
                         ids=["%s-%s-%s" % (c[0], c[1], "x".join(str(a * b) for a, b in
                                                                zip(c[2], c[3]))) for c in TILED])
def test_large_grid_of_copies(lattice, storage, small, copies, what):
    import torch

    from paper_2302_04741_amd import sim

    small = (tuple(small) + (1,))[:3]
    copies = (tuple(copies) + (1,))[:3]
    wl = _fields(lattice, small, 17)
    dims = tuple(a * b for a, b in zip(small, copies))
    dt = {"f64": torch.float64, "f32": torch.float32}[storage]

    def run(d, rho, u, theta):
        s = sim.Sim(lattice, d, wl.tau_hat, rho, u, theta, storage=storage)
        s.set_force(wl.force[1])
        s.step(STEPS)
        h = s.get_populations().view(dt)
        s.close()
        return h

    ref = run(small, wl.rho, wl.u, wl.theta)
    got = run(dims, *(_tile(a, small, copies) for a in (wl.rho, wl.u, wl.theta)))
    q = ref.numel() // (small[0] * small[1] * small[2])
    ref = ref.reshape(q, 1, small[2], 1, small[1], 1, small[0])
    got = got.reshape(q, copies[2], small[2], copies[1], small[1], copies[0], small[0])
    err = float((got - ref).abs().max())
    assert err <= 8 * STEPS * EPS[storage] * float(ref.abs().max())


@pytest.mark.parametrize("lattice,dims,what", [
    ("D3Q39", (120, 120, 120), "end of the sweep kept"),
    ("D3Q39", (160, 144, 144), "end of the sweep kept"),
    ("D2Q37", (2000, 1100), "end of the sweep kept"),
])
def test_f16_sizes_against_fp32(lattice, dims, what):
    from paper_2302_04741_amd import sim

    wl = _fields(lattice, (tuple(dims) + (1,))[:3], 23)
    got = {}
    for storage in ("f32", "f16dev"):
        s = sim.from_workload(wl, storage=storage)
        s.step(STEPS)
        got[storage] = s.moments()
        s.close()
    for a, b, bar in zip(got["f16dev"], got["f32"], (2e-4, 2e-3, 2e-4)):
        assert float((a - b).abs().max()) <= bar * float(b.abs().max())
