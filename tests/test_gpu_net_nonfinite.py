"""An infinity or a NaN in the input of a layer whose output gradient is zero there: zero times it
is NaN and counts in the weight gradient, also where a kernel passes over the steps in which every
output gradient is zero.

Only the last layer (24 -> 3) can show it: its output gradient is the caller's, exactly zero away
from the labelled voxels.  The other layers multiply theirs by GELU'(z), which is NaN wherever the
layer's input is not finite, so there no step with such an input holds zeros alone.

The one nonzero output gradient lies far from the bad sample, so that its own products are finite
and only the products with zero bring the NaN."""
import numpy as np
import pytest
import torch
from scipy.stats import norm

import oracle as O

S, AT = 21, (15, 15, 15)
NW = 3 * 27 * 24  # weights of the last layer


def _case(bad):
    X = np.random.default_rng(3).standard_normal((1, S, S, S)).astype(np.float32)
    X[0, 0, 0, 0] = bad
    dY = np.zeros((1, S, S, S, 3), np.float32)
    dY[(0,) + AT] = (1.0, -2.0, 0.5)
    return X, dY


def _last_input(X, p):
    """Activations entering the last layer."""
    a, o = X[..., None].astype(np.float64), 0
    with np.errstate(invalid="ignore", over="ignore"):
        for ci, co in zip(O.SURROGATE_CHANNELS[:4], O.SURROGATE_CHANNELS[1:5]):
            W = p[o:o + co * 27 * ci].reshape(co, 27, ci)
            z = O.conv3d(a, W, p[o + co * 27 * ci:o + co * 27 * ci + co])
            a, o = z * norm.cdf(z), o + co * 27 * ci + co
    return a


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_case_tells_passed_over_steps_apart(bad):
    """The sums over every voxel are NaN in every weight; those over the voxels with a nonzero
    output gradient alone are finite."""
    X, dY = _case(bad)
    p = np.random.default_rng(1).standard_normal(O.net_num_params()) * 0.1
    a = np.pad(_last_input(X, p)[0], ((1, 1), (1, 1), (1, 1), (0, 0)), mode="reflect")
    every, kept = np.zeros((3, 27, 24)), np.zeros((3, 27, 24))
    for k in range(27):
        t, u, w = k // 9, k // 3 % 3, k % 3
        P = a[t:t + S, u:u + S, w:w + S]
        with np.errstate(invalid="ignore"):
            every[:, k] = np.einsum("tuwc,tuwi->ci", dY[0].astype(np.float64), P)
        kept[:, k] = np.outer(dY[(0,) + AT], P[AT])
    assert np.isnan(every).all() and np.isfinite(kept).all()


@pytest.mark.gpu
@pytest.mark.parametrize("bad", [np.inf, np.nan])
@pytest.mark.parametrize("f32", [True, False])
def test_zero_times_nonfinite_reaches_the_last_layer(bad, f32):
    from paper_1901_11095_amd import sal
    net = sal.Net(seed=5)
    net.set_precision(sal.FP32 if f32 else sal.BF16)
    X, dY = _case(bad)
    Xg = torch.from_numpy(X).cuda()
    net.grads(zero=True)
    net.forward(Xg)
    net.backward(Xg, torch.from_numpy(dY).cuda())
    g = net.grads(zero=True)
    w = g[g.size - NW - 3:g.size - 3]
    assert np.isnan(w).all(), int(np.isnan(w).sum())
    assert np.isfinite(g[g.size - 3:]).all()  # the bias gradient sums the output gradient alone
