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


# sides of the large member: the end of the sweep kept, the same with 8 wavefronts a CU
# in FP32 (the batch of small members alone stays cached)
@pytest.mark.parametrize("storage", ["f32", "f64", "f16dev"])
@pytest.mark.parametrize("lattice,small,sides", [("D2Q37", (200, 150, 1), (1000, 3000)),
                                                 ("D3Q39", (40, 37, 33), (100, 200))])
def test_batch_members_beside_a_large_one_bitwise(lattice, small, sides, storage):
    """The policy follows the bytes of the whole batch and where a tile lies in the
    sweep; a member's result depends on neither: bitwise what it is without the large
    member, before it in the list or after."""
    import torch

    from paper_2302_04741_amd import sim, workloads

    wls = [workloads.random_smooth(lattice, small, seed=3, tau_hat=0.7, force_kind=kind)
           for kind in ("uniform", "axis")]

    def run(members, picked):
        sims = [sim.from_workload(w, storage=storage) for w in members]
        b = sim.Batch(len(sims))
        b.set(sims)
        b.step(STEPS)
        got = [sims[k].get_populations() for k in picked]
        b.close()
        for s in sims:
            s.close()
        return got

    alone = run(wls, (0, 1))
    for n in sides:
        large = (workloads.thermal_shear_2d(n=n) if lattice == "D2Q37"
                 else workloads.kolmogorov_3d(n=n))
        for members, picked in (([wls[0], large, wls[1]], (0, 2)), ([large] + wls, (1, 2))):
            for a, c in zip(alone, run(members, picked)):
                assert torch.equal(a, c), (n, picked)


# members the memory-side cache does not hold, holds one by one, and small ones between
@pytest.mark.parametrize("lattice,storage,sides", [
    ("D2Q37", "f32", (1200, 40, 33, 700, 512, 600, 65)),
    ("D2Q37", "f64", (50, 700, 64, 900, 512, 33)),
    ("D3Q39", "f32", (24, 100, 90, 17, 70, 64)),
    ("D3Q39", "f16dev", (100, 24, 100, 100, 96, 17)),
])
def test_batch_in_groups_equals_step_by_step_bitwise(lattice, storage, sides):
    """Calls of many steps advance a large batch group by group, calls of one step all
    members together: the same states, whoever makes the call."""
    import torch

    from paper_2302_04741_amd import sim, workloads

    steps = 9

    def members():
        return [sim.from_workload(workloads.thermal_shear_2d(n=n) if lattice == "D2Q37"
                                  else workloads.kolmogorov_3d(n=n), storage=storage)
                for n in sides]

    def finish(sims):
        got = [s.get_populations() for s in sims]
        assert all(s.step_count == steps for s in sims)
        for s in sims:
            s.close()
        return got

    sims = members()
    b = sim.Batch(len(sims))
    b.set(sims)
    for _ in range(steps):
        b.step(1)
    b.close()
    want = finish(sims)

    sims = members()
    b = sim.Batch(len(sims))
    b.set(sims)
    b.step(steps)
    b.close()
    for a, c in zip(want, finish(sims)):
        assert torch.equal(a, c)

    sims = members()
    sim.batch_step_noalloc(sims, steps)
    for a, c in zip(want, finish(sims)):
        assert torch.equal(a, c)
