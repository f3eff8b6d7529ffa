"""The empty-space map of the largest volume that a call takes (1625^3 u8, just
below 4 GiB) with the smallest cells: 407^3 of them.  A cell of 8^3 voxels and
the next ones is the union of its eight cells of 4^3, so that map is a minimum
and maximum over this one's; single cells are compared with the voxels."""
import pytest
import torch

from paper_2008_06134_amd import vi

pytestmark = pytest.mark.gpu
DEV = "cuda"


def test_largest_volume_smallest_cells():
    N, cell = 1625, 4
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    raw = torch.empty(N, N, N, dtype=torch.uint8, device=DEV)
    for z in range(0, N, 125):
        # (a range of its own for every part, or most cells would hold 0 and 255)
        raw[z:z + 125] = torch.randint(z // 16, 150 + z // 16, (min(125, N - z), N, N), generator=gen, device=DEV,
                                       dtype=torch.uint8)
    vol = vi.Volume(raw)
    nc = -(-N // cell)
    out = torch.full((nc ** 3 * 2,), -1.0, device=DEV)
    fine = vol.with_minmax(cell, out).minmax.reshape(nc, nc, nc, 2)
    half = -(-N // 8)
    coarse = vol.with_minmax(8).minmax.reshape(half, half, half, 2)
    torch.cuda.synchronize()
    for c, pad in ((0, 2.0), (1, -2.0)):
        p = torch.full((2 * half,) * 3, pad, device=DEV)
        p[:nc, :nc, :nc] = fine[..., c]
        p = p.reshape(half, 2, half, 2, half, 2)
        want = p.amin((1, 3, 5)) if c == 0 else p.amax((1, 3, 5))
        assert torch.equal(want, coarse[..., c])
        del p, want
    scale = torch.tensor(vol.scale, dtype=torch.float32, device=DEV)
    for z, y, x in [(0, 0, 0), (nc - 1, nc - 1, nc - 1), (nc - 1, 0, 17), (0, nc - 1, nc - 1), (203, 99, 301), (406, 200, 5)]:
        s = raw[4 * z:4 * z + 5, 4 * y:4 * y + 5, 4 * x:4 * x + 5].float() * scale
        assert torch.equal(fine[z, y, x], torch.stack([s.min(), s.max()])), (z, y, x)
