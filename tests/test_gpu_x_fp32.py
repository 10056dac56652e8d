"""FP32 X-engine (its products are sums of BF16 products): accuracy against
64 bits over signal counts at the edges of its tiles, step counts and splits,
over the exponent range, and with cells that are not finite.

Bound on a visibility's error, relative to sqrt(V_ii V_jj): each product is
exact to 2^-24 of |a b| (three dropped terms of at most 2^-26 each), each
matrix instruction rounds its sum of at most 32 terms (6 of them per 16
spectra, counted at 2^-23), and the running sum rounds once per 16 spectra."""
import numpy as np
import pytest

import paper_0910_1517_amd as corr
import synth
from gpu_util import pack_input

pytestmark = pytest.mark.gpu


def visibilities(Y, x_split=0):
    import torch
    S, T, C, _ = Y.shape
    plan = corr.Plan(S, 2 * C, T, precision=corr.FP32, x_split=x_split)
    spec = pack_input(plan, Y)
    acc, state, vis = plan.alloc("acc"), plan.alloc("state"), plan.alloc("vis")
    plan.xengine(spec, acc)
    plan.integrate(acc, state, vis, None, flags=corr.DUMP)
    torch.cuda.synchronize()
    st = state.cpu().numpy().reshape(C, -1, 2)
    return st[..., 0], st[..., 1]


def reference(Y):
    y = Y[..., 0].astype(np.float64) + 1j * Y[..., 1]
    S = y.shape[0]
    j, i = np.tril_indices(S)
    V = np.einsum("smk,tmk->kst", y, y.conj(), optimize=True)
    p = np.sqrt(np.einsum("kss->ks", V).real)
    return V[:, i, j], p[:, i] * p[:, j]


@pytest.mark.parametrize("S,T,x_split", [(1, 32, 1), (2, 64, 1), (31, 32, 1), (32, 96, 3), (33, 32, 1), (48, 96, 1),
                                         (63, 160, 5), (64, 64, 2), (64, 1024, 1)])
def test_accuracy(S, T, x_split):
    C = 256
    g = synth.rng(S * 1000 + T, 51)
    Y = (g.standard_normal((S, T, C, 2)) + 0.5 * g.standard_normal((1, T, C, 2))).astype(np.float32)
    Y *= np.float32(10.0) ** g.integers(-12, 13, (1, 1, C, 1)).astype(np.float32)  # the channels' scales
    re, im = visibilities(Y, x_split)
    V, scale = reference(Y)
    tol = 2.0 ** -24 * (8 + T / 16)
    err = np.abs(re + 1j * im - V) / scale
    print("S=%d T=%d: max error %.3g of the pair's power, bound %.3g" % (S, T, err.max(), tol))
    assert err.max() <= tol


@pytest.mark.parametrize("S", [20, 50])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38])
def test_cells_that_are_not_finite(S, value):
    """A bad cell spoils its own signal's pairs in its own channel, and only them."""
    T, C, s, k = 64, 256, 13, 77
    Y = synth.rng(S, 52).standard_normal((S, T, C, 2)).astype(np.float32)
    Y[s, 40, k, 0] = value
    Y[s, 40, k, 1] = 0.0
    re, im = visibilities(Y)
    with np.errstate(all="ignore"):
        V, scale = reference(np.where(np.abs(Y) < 1e30, Y, 0))
    j, i = np.tril_indices(S)
    bad = np.zeros(re.shape, bool)
    bad[k] = (i == s) | (j == s)
    with np.errstate(invalid="ignore"):
        good = np.abs(re + 1j * im - V) <= 2.0 ** -24 * (8 + T / 16) * scale
    assert good[~bad].all()
    assert not good[bad].any()
    auto = re[k, (i == s) & (j == s)][0]
    assert np.isnan(auto) if np.isnan(value) else auto == np.inf
    if value == 3.4e38:  # of its products with other signals, those that FP32 holds are there
        full = reference(Y[:, :, k:k + 1])[0][0].real
        pairs = bad[k] & (i != j)
        held = np.abs(full[pairs]) < np.finfo(np.float32).max
        assert np.array_equal(np.isfinite(re[k, pairs]), held)
        assert np.abs(re[k, pairs][held] / full[pairs][held] - 1).max() <= 2.0 ** -24 * (8 + T / 16)
