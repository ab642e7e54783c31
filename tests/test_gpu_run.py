"""Cubes 9..15 and 17..20 with overlapping windows: the kernel that shares the first two
stages along a run of windows (k_energy_run) against the one that takes a window at a time
(k_energy_win).  Both do the same arithmetic in the same order, so where they compute the same
window the energies are equal bit for bit: a non-overlapping lattice (stride L) runs window by
window and its lattice voxels hold the windows' own energies (interpolation weight zero).
The widths put run tails of one window, and runs cut to 8 and 16, under test.
"""
import pytest
import torch

from paper_1901_11095_amd import sal, synth

pytestmark = pytest.mark.gpu


def energies(L, V, stride):
    _, E, _, _ = sal.Saliency(L=L, stride=stride).saliency_maps(V)
    return E


@pytest.mark.parametrize("L", [9, 10, 11, 12, 13, 14, 15, 17, 18, 19, 20])
@pytest.mark.parametrize("shape", [(23, 41, 65), (22, 21, 33), (70, 64, 41)])
def test_runs_equal_single_windows(L, shape):
    print("runs L=%d shape %s" % (L, shape), flush=True)
    V = torch.from_numpy(synth.make_volume(shape, seed=L, n_faults=1, throw=2)).cuda()
    one = energies(L, V, L)[:, ::L, ::L, ::L]
    assert torch.equal(energies(L, V, 1)[:, ::L, ::L, ::L], one)


@pytest.mark.parametrize("L,stride", [(9, 2), (9, 4), (11, 5), (12, 3), (13, 6), (17, 8), (20, 2), (20, 5), (20, 9)])
def test_strided_runs_equal_single_windows(L, stride):
    """On the lattices of overlapping strides (at cube 20 the widest fall back to single
    windows) against the windows at every voxel."""
    V = torch.from_numpy(synth.make_volume((45, 38, 83), seed=L + stride, n_faults=1, throw=2)).cuda()
    a = energies(L, V, stride)[:, ::stride, ::stride, ::stride]
    assert torch.equal(a, energies(L, V, 1)[:, ::stride, ::stride, ::stride])


def test_box_and_batch_equal_whole_volume():
    L, shape = 12, (44, 50, 61)
    V = torch.from_numpy(synth.make_volume(shape, seed=3, n_faults=1, throw=2)).cuda()
    ctx = sal.Saliency(L=L)
    _, _, Sr, st = ctx.saliency_maps(V)
    for lo, dims in [((0, 0, 0), (5, 7, 9)), ((20, 11, 28), (24, 39, 33))]:
        sl = (slice(None),) + tuple(slice(a, a + d) for a, d in zip(lo, dims))
        assert torch.equal(ctx.raw_box(V, lo, dims), Sr[sl])
    tiles, td = [(0, 0, 0), (30, 42, 53), (12, 20, 8)], (14, 8, 8)
    X = torch.empty((len(tiles), 3) + td, dtype=torch.float32, device="cuda")
    err = torch.zeros(len(tiles), dtype=torch.float32, device="cuda")
    sal.check_tiles(ctx, V, tiles, Sr.clone(), tiles, td, st, 0.02, err, exact_out=X)
    for k, lo in enumerate(tiles):
        sl = (slice(None),) + tuple(slice(a, a + d) for a, d in zip(lo, td))
        assert torch.equal(X[k], Sr[sl]), lo


@pytest.mark.parametrize("L,stride", [(9, 1), (10, 4), (12, 3), (18, 1), (20, 2)])
def test_batch_of_one_and_of_two(L, stride):
    """A lone tile takes as many workgroups as it has runs, a tile of a larger batch at most 64 (each
    with several runs): both equal the box of the same voxels bit for bit."""
    shape, td = (60, 61, 63), (26, 30, 33)
    V = torch.from_numpy(synth.make_volume(shape, seed=L, n_faults=1, throw=2)).cuda()
    ctx = sal.Saliency(L=L, stride=stride)
    _, _, Sr, st = ctx.saliency_maps(V)
    for tiles in ([(17, 15, 14)], [(0, 31, 30), (17, 15, 14)]):
        X = torch.empty((len(tiles), 3) + td, dtype=torch.float32, device="cuda")
        err = torch.zeros(len(tiles), dtype=torch.float32, device="cuda")
        sal.check_tiles(ctx, V, tiles, Sr.clone(), tiles, td, st, 0.02, err, exact_out=X)
        for k, lo in enumerate(tiles):
            assert torch.equal(X[k], ctx.raw_box(V, lo, td)), (len(tiles), lo)
