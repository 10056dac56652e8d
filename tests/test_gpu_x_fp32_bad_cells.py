"""FP32 X-engine with cells that are not finite, in its masked and gated forms as well:
such a block is done on the FP32 instructions, found in its first spectra, after a span
of them or at its end.  Signal counts of one tile, of one signal in the second tile
(whose waves mostly have no signal to load) and of two nearly full ones.  The values
are small integers, whose sums are exact in FP32 in any order and on both paths: every
sum that a bad cell has no part in is the exact one."""
import numpy as np
import pytest

import paper_0910_1517_amd as corr
import synth
from gpu_util import pack_input

pytestmark = pytest.mark.gpu
T, C, BAD_S, BAD_K = 1024, 256, 13, 77
SIGNALS = [20, 33, 50]
PLACES = [0, 9, 300, T - 1]  # spectrum of the bad cell


def data(S):
    return synth.rng(S, 91).integers(-4, 5, (S, T, C, 2)).astype(np.float32)


def exact(Y, weight=None):
    """Sums of the pairs [C][P][2]; weight: of each spectrum, 0 or 1."""
    import torch
    y = torch.from_numpy(Y).cuda().permute(2, 0, 1, 3).double()  # [C][S][T][2]
    w = y if weight is None else y * torch.from_numpy(weight.astype(np.float64)).cuda()[:, None]
    r, q, rw, qw = y[..., 0], y[..., 1], w[..., 0], w[..., 1]
    dot = lambda a, b: torch.bmm(a.contiguous(), b.transpose(1, 2).contiguous())
    j, i = np.tril_indices(Y.shape[0])
    re, im = dot(r, rw) + dot(q, qw), dot(q, rw) - dot(r, qw)  # V[i][j] = sum y_i conj(y_j)
    return torch.stack([re[:, i, j], im[:, i, j]], -1).float().cpu().numpy()


def plan_for(S):
    return corr.Plan(S, 2 * C, T, precision=corr.FP32, x_split=1)


def sums(plan, acc):
    return acc.view(plan.C, plan.P, 2).cpu().numpy()


def x(plan, Y, keep=None):
    acc = plan.alloc("acc")
    plan.xengine(pack_input(plan, Y), acc, keep=keep)
    return sums(plan, acc)


def pairs_of(S, s):
    j, i = np.tril_indices(S)
    return (i == s) | (j == s)


def keep_words(plan, S, flags):
    """flags: bool [S][T][C]."""
    import torch
    keep = plan.alloc("keep", zero=False)
    plan.apply_flags(torch.from_numpy(flags.astype(np.uint8)).cuda(), None, keep)
    return keep


def spoils_its_own_pairs_only(got, clean, S):
    own = np.zeros(clean.shape, bool)
    own[BAD_K, pairs_of(S, BAD_S)] = True
    assert not np.isfinite(got[own]).all()
    assert np.array_equal(got[~own], clean[~own])


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("m", PLACES)
@pytest.mark.parametrize("S", SIGNALS)
def test_masked(S, m, value):
    """A bad cell that is flagged is as a cell of zeros, bit for bit; one that is not spoils
    its own pairs."""
    Y = data(S)
    flags = synth.rng(S + m, 92).random((S, T, C)) < 0.05
    zeroed = np.where(flags[..., None], np.float32(0), Y)
    plan = plan_for(S)
    for flagged in (True, False):
        flags[BAD_S, m, BAD_K] = flagged
        zeroed[BAD_S, m, BAD_K] = 0 if flagged else Y[BAD_S, m, BAD_K]
        bad = Y.copy()
        bad[BAD_S, m, BAD_K, 0] = value
        got, clean = x(plan, bad, keep_words(plan, S, flags)), exact(zeroed)
        if flagged:
            assert np.array_equal(got, clean)
        else:
            spoils_its_own_pairs_only(got, clean, S)


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("m", PLACES)
@pytest.mark.parametrize("S", SIGNALS)
def test_gated(S, m, value):
    import torch
    Y, plan, bins = data(S), plan_for(S), 3
    gate = synth.rng(S + m, 93).integers(0, bins, T).astype(np.uint8)
    bad = Y.copy()
    bad[BAD_S, m, BAD_K, 0] = value

    acc = torch.zeros(bins, plan.acc_bytes // 4, device="cuda")
    plan.xengine_gated(pack_input(plan, bad), torch.from_numpy(gate).cuda(), bins, acc)
    spoils_its_own_pairs_only(sums(plan, acc[gate[m]]), exact(Y, gate == gate[m]), S)


@pytest.mark.parametrize("form", ["plain", "masked", "gated"])
@pytest.mark.parametrize("first", [0, 260])
@pytest.mark.parametrize("S", SIGNALS)
def test_dead_antenna(S, first, form):
    """NaN throughout, or from some spectrum on: all and only its own pairs are NaN."""
    import torch
    Y, plan = data(S), plan_for(S)
    flags = np.zeros((S, T, C), bool)
    flags[:, 4::7] = True
    kept = np.where(flags[..., None], np.float32(0), Y) if form == "masked" else Y
    want = [exact(kept, np.arange(T) % 2 == b) for b in range(2)] if form == "gated" else [exact(kept)]
    Y[BAD_S, first:] = np.nan
    if form == "gated":
        acc = torch.zeros(2, plan.acc_bytes // 4, device="cuda")
        plan.xengine_gated(pack_input(plan, Y), (torch.arange(T) % 2).to(torch.uint8).cuda(), 2, acc)
        got = [sums(plan, a) for a in acc]
    else:
        got = [x(plan, Y, keep_words(plan, S, flags) if form == "masked" else None)]
    own = pairs_of(S, BAD_S)
    for g, w in zip(got, want):
        assert np.array_equal(g[:, ~own], w[:, ~own])
        assert np.isnan(g[:, own, 0]).all()
