"""Initial states of large grids by the number of wavefronts a row: how many blocks share
a compute unit follows from it (F16 rows of 5 wavefronts fit three), the values do not.
The moments at step 0 are the fields handed in, and rebuilt for a force they stay so."""
import pytest

pytestmark = pytest.mark.gpu

# rounding of a state at rest density 1: a few units of the storage's precision in the
# sums of 39 populations (F16 rounds the initial state to nearest, 2^-11 of a deviation of
# a few hundredths)
TOL = {"f32": 2e-6, "f16dev": 2e-4}


@pytest.mark.parametrize("storage,nx,rows", [
    ("f16dev", 300, (240, 240)), ("f16dev", 320, (240, 230)), ("f16dev", 500, (180, 180)),
    ("f32", 300, (100, 96)), ("f32", 440, (80, 80)), ("f32", 500, (80, 70)),
])
def test_initial_state_by_wavefronts_a_row(storage, nx, rows):
    import torch

    from paper_2302_04741_amd import sim, workloads

    wl = workloads.random_smooth("D3Q39", (nx,) + rows, seed=4, g_amp=1e-4)
    s = sim.Sim("D3Q39", wl.dims, wl.tau_hat, wl.rho, wl.u, wl.theta, storage=storage)
    want = [torch.from_numpy(a).cuda() for a in (wl.rho, wl.u, wl.theta)]
    for _ in range(2):
        for got, exact in zip(s.moments(), want):
            assert float((got - exact).abs().max()) <= TOL[storage]
        s.set_force(wl.force[1])
    s.close()
