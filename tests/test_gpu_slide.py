"""Cube 8 and 16 in FP32 with the windows sliding along t (k_energy_slide) against the oracle,
for windows at every voxel and on the lattices of the strides below L/2.

Each window's spectrum is the previous window's plus the 2-D DFT of the entering minus the
leaving t-plane; the running sums restart at the windows t0 = 0, L/2 and every multiple of 512.
A volume of 560 rows spans all three kinds of segment (and 10 x 19 positions a ragged y
tile): E, the raw maps and S within 1e-5 of each map's maximum against the FP64 oracle, and
within 1e-6 of the kernel that contracts every window along t on its own.  Boxes and batched
tile checks whose rows straddle the restarts equal the whole-volume maps bit for bit (the
segments are fixed rows of the volume, so a window's arithmetic does not depend on the box).
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1901_11095_amd import sal, synth

pytestmark = pytest.mark.gpu

SHAPE = (560, 10, 19)


def relmax(got, ref):
    got, ref = np.asarray(got, np.float64), np.asarray(ref, np.float64)
    return float(np.abs(got - ref).max() / max(np.abs(ref).max(), 1e-300))


@pytest.fixture(scope="module")
def volume():
    return synth.make_volume(SHAPE, seed=31, n_faults=2, throw=3, n_chaotic=1, chaotic_size=8)


@pytest.fixture(scope="module", params=[8, 16])
def maps(volume, request):
    L = request.param
    ctx = sal.Saliency(L=L)
    Vd = torch.from_numpy(volume).cuda()
    S, E, Sr, st = ctx.saliency_maps(Vd)
    torch.cuda.synchronize()
    return ctx, Vd, S.cpu().numpy(), E.cpu().numpy(), Sr.cpu().numpy(), st.cpu().numpy()


def test_slide_vs_oracle(volume, maps):
    ctx, _, S, E, Sr, _ = maps
    print("sliding cube %d on %s vs oracle" % (ctx.L, SHAPE), flush=True)
    ref = O.saliency(volume, O.Params(L=ctx.L))
    for m in range(3):
        assert relmax(E[m], ref["E"][m]) <= 1e-5, ("E", m, relmax(E[m], ref["E"][m]))
        assert relmax(Sr[m], ref["S_raw"][m]) <= 1e-5, ("S_raw", m, relmax(Sr[m], ref["S_raw"][m]))
    assert np.abs(S - ref["S"]).max() <= 1e-5


def test_slide_vs_direct(volume, maps):
    ctx, Vd, _, E, _, _ = maps
    cd = sal.Saliency(L=ctx.L, t_direct=True)
    assert cd.params.t_direct == 1
    _, Ed, _, _ = cd.saliency_maps(Vd)
    Ed = Ed.cpu().numpy()
    for m in range(3):
        assert relmax(E[m], Ed[m]) <= 1e-6, (m, relmax(E[m], Ed[m]))


@pytest.mark.parametrize("lo,dims", [((506, 0, 3), (12, 10, 16)), ((2, 5, 0), (10, 5, 19)),
                                     ((511, 9, 18), (49, 1, 1)), ((0, 0, 0), (560, 3, 17))])
def test_slide_boxes_equal_whole_volume(maps, lo, dims):
    ctx, Vd, _, _, Sr, _ = maps
    box = ctx.raw_box(Vd, lo, dims).cpu().numpy()
    sl = (slice(None),) + tuple(slice(a, a + d) for a, d in zip(lo, dims))
    assert np.array_equal(box, Sr[sl])


def test_slide_batch_equals_whole_volume(maps):
    ctx, Vd, _, _, Sr, st = maps
    tiles = [(504, 0, 0), (0, 2, 5), (20, 0, 11), (544, 2, 11), (120, 2, 0)]
    td = (16, 8, 8)
    P = torch.from_numpy(Sr).cuda() + 1.0  # every tile over the bound: replaced by the exact maps
    X = torch.empty((len(tiles), 3) + td, dtype=torch.float32, device="cuda")
    err = torch.zeros(len(tiles), dtype=torch.float32, device="cuda")
    sal.check_tiles(ctx, Vd, tiles, P, tiles, td, torch.from_numpy(st).cuda(), 0.02, err, exact_out=X)
    torch.cuda.synchronize()
    X, P = X.cpu().numpy(), P.cpu().numpy()
    for k, lo in enumerate(tiles):
        sl = (slice(None),) + tuple(slice(a, a + d) for a, d in zip(lo, td))
        assert np.array_equal(X[k], Sr[sl]), lo
        assert np.array_equal(P[sl], Sr[sl]), lo


@pytest.mark.parametrize("L", [8, 16])
def test_slide_invariants(L):
    """The invariants the oracle's pins fix, on the sliding kernel: a constant volume has no
    energy outside DC and zero saliency; adding a constant changes no energy; exchanging t and
    x exchanges E_t and E_x (t slides, x is contracted directly, so the two axes go through
    different arithmetic)."""
    ctx = sal.Saliency(L=L)
    C = np.full((36, 40, 37), 2.5, np.float32)
    S, E, _, _ = ctx.saliency_maps(torch.from_numpy(C).cuda())
    assert float(E.abs().max()) <= 1e-6 * 2.5
    assert bool(torch.all(S == 0))
    V = synth.make_volume((36, 40, 37), seed=17, n_faults=1, throw=3, n_chaotic=1, chaotic_size=8)
    _, E0, S0, _ = ctx.saliency_maps(torch.from_numpy(V).cuda())
    _, E1, S1, _ = ctx.saliency_maps(torch.from_numpy(V + 3.0).cuda())
    assert relmax(E1.cpu().numpy(), E0.cpu().numpy()) <= 1e-5
    assert relmax(S1.cpu().numpy(), S0.cpu().numpy()) <= 1e-5
    Vp = np.ascontiguousarray(V.transpose(1, 0, 2))
    _, Ep, _, _ = ctx.saliency_maps(torch.from_numpy(Vp).cuda())
    E0, Ep = E0.cpu().numpy(), Ep.cpu().numpy()
    for m, mp in [(0, 1), (1, 0), (2, 2)]:
        assert relmax(Ep[mp], E0[m].transpose(1, 0, 2)) <= 1e-5, m


@pytest.fixture(scope="module", params=[(8, 2), (8, 3), (16, 2), (16, 3), (16, 4), (16, 7)])
def maps2(volume, request):
    """Windows on the stride-s lattice: the sums slide one row per step, the magnitudes are
    taken at every s-th window."""
    L, st = request.param
    ctx = sal.Saliency(L=L, stride=st)
    Vd = torch.from_numpy(volume).cuda()
    S, E, Sr, st = ctx.saliency_maps(Vd)
    torch.cuda.synchronize()
    return ctx, Vd, S.cpu().numpy(), E.cpu().numpy(), Sr.cpu().numpy()


def test_slide_strided_vs_oracle(volume, maps2):
    ctx, _, S, E, Sr = maps2
    st = ctx.params.stride
    print("sliding cube %d stride %d on %s vs oracle" % (ctx.L, st, SHAPE), flush=True)
    ref = O.saliency(volume, O.Params(L=ctx.L, stride=st))
    for m in range(3):
        assert relmax(E[m], ref["E"][m]) <= 1e-5, ("E", m, relmax(E[m], ref["E"][m]))
        assert relmax(Sr[m], ref["S_raw"][m]) <= 1e-5, ("S_raw", m, relmax(Sr[m], ref["S_raw"][m]))
    assert np.abs(S - ref["S"]).max() <= 1e-5


def test_slide_strided_vs_direct(maps2):
    """Against the kernels that contract every window along t on its own (the fused kernel at
    stride 2, the window-by-window kernel above)."""
    ctx, Vd, _, E, _ = maps2
    cd = sal.Saliency(L=ctx.L, stride=ctx.params.stride, t_direct=True)
    _, Ed, _, _ = cd.saliency_maps(Vd)
    Ed = Ed.cpu().numpy()
    for m in range(3):
        assert relmax(E[m], Ed[m]) <= 1e-6, (m, relmax(E[m], Ed[m]))


@pytest.mark.parametrize("lo,dims", [((500, 1, 3), (20, 8, 16)), ((2, 5, 0), (10, 5, 19)),
                                     ((511, 9, 18), (49, 1, 1))])
def test_slide_strided_boxes_equal_whole_volume(maps2, lo, dims):
    ctx, Vd, _, _, Sr = maps2
    box = ctx.raw_box(Vd, lo, dims).cpu().numpy()
    sl = (slice(None),) + tuple(slice(a, a + d) for a, d in zip(lo, dims))
    assert np.array_equal(box, Sr[sl])


@pytest.mark.parametrize("L,stride", [(8, 1), (8, 3), (16, 1), (16, 5)])
@pytest.mark.parametrize("rows", [39, 128])
def test_small_volumes_in_parts(L, stride, rows):
    """Few columns: a segment's windows are split over workgroups that repeat the earlier
    updates (up to eight parts, the last ones short or empty).  Against the oracle, and bit for
    bit equal to the same rows of boxes that take other parts of the walk."""
    V = synth.make_volume((rows, 11, 18), seed=rows + L, n_faults=1, throw=3)
    ctx = sal.Saliency(L=L, stride=stride)
    Vd = torch.from_numpy(V).cuda()
    S, E, Sr, st = ctx.saliency_maps(Vd)
    ref = O.saliency(V, O.Params(L=L, stride=stride))
    for m in range(3):
        assert relmax(E[m].cpu().numpy(), ref["E"][m]) <= 1e-5, m
    assert float(st[6]) == float(np.abs(V).max())
    for lo, d in ((0, 3), (L // 2 - 1, 5), (17, 12), (rows - 7, 7)):
        box = ctx.raw_box(Vd, (lo, 1, 2), (d, 9, 15))
        assert torch.equal(box, Sr[:, lo:lo + d, 1:10, 2:17]), lo
