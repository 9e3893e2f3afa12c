"""A run between plates resumes bitwise from its populations and step count: the pass
that forms the plates' sums of an imported state gives the bits that the step which
produced the state had given (rows shared by both plates, ny < 3, included)."""
import pytest

from paper_2302_04741_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
@pytest.mark.parametrize("lattice,nx,nz", [("D2Q37", 70, 1), ("D3Q39", 9, 5)])
@pytest.mark.parametrize("ny", [1, 2, 3, 5, 19])
def test_resume_between_plates_is_bitwise(lattice, nx, nz, ny, storage):
    import torch

    from paper_2302_04741_amd import sim

    def make(seed):
        wl = workloads.random_smooth(lattice, (nx, ny, nz), seed=seed, g_amp=2e-4, amp_u=0.03)
        wl.walls = (0.9, 1.2, 0.02, -0.03)
        return sim.from_workload(wl, storage=storage)

    a, b = make(1), make(1)
    a.step(7)
    saved = a.get_populations()
    a.step(6)
    b.step(2)  # another state and other sums, replaced below
    b.set_populations(saved)
    b.step_count = 7
    b.step(6)
    assert torch.equal(a.get_populations(), b.get_populations())
    a.close()
    b.close()
