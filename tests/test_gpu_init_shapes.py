"""The initial state over the launch shapes of its kernels (blocks of whole rows of 1 to
8 wavefronts, split rows beyond, small and large grids): the moments reported at step 0
are the fields handed in, at creation and after a force was set.

Tolerance: a moment is a sum of 37 or 39 values of at most about 0.3 in deviation form,
each rounded once: 40 * 0.3 eps, and twice that for theta (a quotient of two of them) and
for the rebuilt state: 40 eps."""
import pytest

pytestmark = pytest.mark.gpu

EPS = {"f64": 2.0 ** -53, "f32": 2.0 ** -24}

SHAPES = [("D2Q37", (nx, ny)) for nx, ny in
          ((1, 5), (63, 4), (65, 3), (129, 7), (193, 5), (257, 3), (321, 6), (385, 3), (449, 5),
           (512, 3), (513, 3), (577, 2), (1025, 3), (65, 2100), (200, 1100), (450, 700),
           (600, 480))]
SHAPES += [("D3Q39", d) for d in ((70, 5, 3), (129, 40, 36), (200, 33, 40), (500, 20, 21))]


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("lattice,dims", SHAPES + [("D3Q39", (160, 160, 144)),
                                                   ("D2Q37", (1700, 1700))])
def test_initial_moments_are_the_inputs(lattice, dims, storage):
    import torch

    from paper_2302_04741_amd import sim, workloads

    wl = workloads.random_smooth(lattice, (tuple(dims) + (1,))[:3], seed=5)
    want = [torch.as_tensor(a).cuda() for a in (wl.rho, wl.u, wl.theta)]
    s = sim.Sim(lattice, dims, wl.tau_hat, *want, storage=storage)

    def check():
        for got, ref in zip(s.moments(), want):
            assert float((got - ref).abs().max()) <= 40 * EPS[storage] * 1.2

    check()
    s.set_force(wl.force[1])     # rebuilds the state with the force
    check()
    prof = torch.ones((s.D, s.dims[1]), dtype=torch.float64)
    s.set_force(axis=1, profile=prof * torch.as_tensor(wl.force[1])[:, None])
    check()
    s.set_force([0.0] * len(wl.force[1]))  # from a table: through the fields
    check()
    assert s.step_count == 0
    s.close()
