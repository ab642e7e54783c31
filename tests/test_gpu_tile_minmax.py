"""Extremes of the raw maps per tile (sal_tile_minmax) against torch, bit for bit: tiles of one
voxel, tiles on both sides of the size from which a tile takes more waves (2^14 voxels: sides 25 and
26, and a flat volume), tiles past the volume, ragged edges, infinities and NaN.  The running minimum
starts at the largest float and the running maximum at the lowest, so a tile of +inf alone reports
the largest float as its minimum."""
import pytest
import torch

from paper_1901_11095_amd import sal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,tile", [((7, 9, 11), 1), ((13, 10, 21), 2), ((40, 41, 43), 8),
                                        ((60, 55, 53), 25), ((60, 55, 53), 26), ((9, 70, 90), 42),
                                        ((9, 70, 90), 43), ((30, 31, 33), 1024)])
@pytest.mark.parametrize("bad", [None, float("nan"), float("inf"), -float("inf")])
def test_tile_extremes(shape, tile, bad):
    g = torch.Generator().manual_seed(tile)
    M = torch.randn((3,) + shape, generator=g)
    if bad is not None:
        M[0, 3, 4, 5] = M[2, -1, -1, -1] = bad
    out = sal.tile_minmax(sal.Saliency(L=5), M.cuda(), tile).cpu()
    ref = []
    for t in range(0, shape[0], tile):
        for x in range(0, shape[1], tile):
            for y in range(0, shape[2], tile):
                c = M[:, t:t + tile, x:x + tile, y:y + tile].reshape(3, -1)
                lo, hi = c.min(dim=1).values, c.max(dim=1).values
                lo, hi = lo.clamp(max=torch.finfo(torch.float32).max), hi.clamp(min=torch.finfo(torch.float32).min)
                nan = c.isnan().any(dim=1)
                lo[nan], hi[nan] = -float("inf"), float("inf")
                ref.append(torch.stack([lo, hi], dim=1).flatten())
    assert torch.equal(out, torch.stack(ref))
