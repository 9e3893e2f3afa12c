"""Results do not depend, bit for bit, on the width of the blocks.

Single grids larger than the memory-side cache: the width moves the line between the part
of a sweep whose stores are streamed and the part whose stores are kept, which are two
compilations of the same update; the default of each size is one of the widths."""
import pytest

pytestmark = pytest.mark.gpu

CASES = [
    ("D2Q37", "f32", (1100, 1000, 1)),    # the end of each sweep kept
    ("D2Q37", "f32", (1801, 1600, 1)),    # the same, 8 wavefronts a CU
    ("D2Q37", "f64", (901, 800, 1)),
    ("D2Q37", "f16dev", (1900, 1501, 1)),
    ("D3Q39", "f32", (150, 120, 100)),
    ("D3Q39", "f64", (101, 95, 90)),      # non-temporal loads
    ("D3Q39", "f64", (193, 125, 150)),    # 1 GiB and more: 256 threads, 8 wavefronts a CU
    ("D3Q39", "f16dev", (250, 240, 235)),  # 1 GiB and more: 512 threads
]


@pytest.mark.parametrize("lattice,storage,dims", CASES)
def test_every_width_gives_the_same_bits(lattice, storage, dims):
    import torch

    from paper_2302_04741_amd import sim, workloads

    wl = workloads.random_smooth(lattice, dims, seed=9, tau_hat=0.7)
    s = sim.from_workload(wl, storage=storage)
    first = s.get_populations()
    want = None
    for threads in (0, 64, 128, 256) + ((512, 1024) if storage != "f64" else ()):
        s.set_populations(first)
        s.step_count = 0
        s.set_block(threads)
        s.step(3)
        got = s.get_populations()
        if want is None:
            want = got
        else:
            assert torch.equal(got, want), threads
    s.close()


# tiles of the FP64 lists around the lines between which the default is 256 threads
@pytest.mark.parametrize("sides", [(64,) * 7, (64,) * 7 + (2,), (52, 162), (64,) * 11,
                                   (64,) * 11 + (2,)])
def test_batch_default_width_gives_the_same_bits(sides):
    import torch

    from paper_2302_04741_amd import sim, workloads

    got = []
    for threads in (0, 64, 128, 256):
        sims = [sim.from_workload(workloads.thermal_shear_2d(n=n), storage="f64") for n in sides]
        b = sim.Batch(len(sims))
        b.set(sims)
        if threads:
            b.set_launch(threads, 0)
        b.step(3)
        got.append([s.get_populations() for s in sims])
        b.close()
        for s in sims:
            s.close()
    for other in got[1:]:
        assert all(torch.equal(a, c) for a, c in zip(got[0], other))
