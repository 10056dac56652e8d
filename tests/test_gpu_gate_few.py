"""Gated FP32 X-engine with few spectra in a gate: each rounds no more than FP32 products
added one after the other do.  Of n spectra, a real part is 2 n products and as many
additions of the running sum, each exact to 2^-24 of it, and the sum never exceeds the
pair's power p = sqrt(V_ii V_jj): 2 n 2^-24 p.  An imaginary part is two such sums of n
products, which together never exceed p, and their difference: (n + 1) 2^-24 p at most."""
import numpy as np
import pytest

import paper_0910_1517_amd as corr
import synth
from gpu_util import acc_sum, pack_input

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [7, 32, 33, 64])
@pytest.mark.parametrize("n", [0, 1, 2, 4, 5])
@pytest.mark.parametrize("T,x_split", [(32, 1), (2048, 2)])
def test_roundings(S, n, T, x_split):
    import torch
    C, bins = 256, 3
    g = synth.rng(S * 10 + n, 94)
    Y = g.standard_normal((S, T, C, 2)).astype(np.float32)
    gate = np.full(T, 2, np.uint8)
    at = g.choice(T // x_split, n, replace=False) + (T - T // x_split)  # all in the last split
    gate[at] = 1
    plan = corr.Plan(S, 2 * C, T, precision=corr.FP32, x_split=x_split)
    assert plan.splits == x_split
    acc = torch.zeros(bins, plan.acc_bytes // 4, device="cuda")
    plan.xengine_gated(pack_input(plan, Y), torch.from_numpy(gate).cuda(), bins, acc)
    got = acc_sum(acc[1].cpu().numpy(), plan)
    y = Y[:, at].astype(np.float64)
    y = (y[..., 0] + 1j * y[..., 1]).transpose(2, 0, 1)  # [C][S][n]
    V = y @ y.conj().transpose(0, 2, 1)
    j, i = np.tril_indices(S)
    p = np.sqrt(np.einsum("kss->ks", V).real)
    scale, V = p[:, i] * p[:, j], V[:, i, j]
    if n == 0:
        assert not got.any()
    elif n <= 4:
        assert np.all(np.abs(got[..., 0] - V.real) <= 2 * n * 2.0 ** -24 * scale)
        assert np.all(np.abs(got[..., 1] - V.imag) <= (n + 1) * 2.0 ** -24 * scale)
    else:
        assert np.abs(got[..., 0] + 1j * got[..., 1] - V).max() <= (2.0 ** -24 * (8 + T / 16) * scale).max()
