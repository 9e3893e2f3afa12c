"""The server's copy of kept results into host memory (two pinned buffers taken in
turn): bit for bit at sizes around one and several pieces, one copier used repeatedly,
and results that do not share memory with each other."""
import pytest

pytestmark = pytest.mark.gpu


def test_pieces_bit_for_bit():
    import torch

    from paper_2302_04741_amd import serve

    copy = serve._HostCopy()
    p = copy.PIECE
    gen = torch.Generator(device="cuda").manual_seed(3)
    results = []
    for n in (0, 1, 4095, p - 1, p, p + 1, 2 * p, 3 * p + 5):
        src = torch.randint(0, 256, (n,), dtype=torch.uint8, device="cuda", generator=gen)
        out = copy(src)
        assert out.device.type == "cpu" and not out.is_pinned()
        results.append((out, src))
    for out, src in results:  # none overwritten by a later copy
        assert torch.equal(out, src.cpu())
