"""Gated X-engine on both sides of its rule for pairs of bins (K-steps a split, odd and
even bin counts, signal counts): each bin's sums, added to what the accumulator held,
are the exact ones of that bin's spectra."""
import numpy as np
import pytest

import paper_0910_1517_amd as corr
import synth
from gpu_util import acc_sum, pack_input

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["int8", "e4m3"])
@pytest.mark.parametrize("T,x_split", [(64, 2), (64, 1), (512, 2)])  # one, two and eight K-steps a split
@pytest.mark.parametrize("bins", [2, 3, 5, 8, 9])
@pytest.mark.parametrize("S", [1, 8, 9, 20, 21, 32, 33])
def test_every_bin(S, bins, T, x_split, prec):
    import torch
    N = 512
    P = {"int8": corr.INT8, "e4m3": corr.FP8_E4M3}[prec]
    g = synth.rng(100 * S + bins + T, 62)
    v = g.integers(-4, 5, (S, T, N // 2, 2))
    if prec == "int8":
        Y = v.astype(np.int8)
    else:  # small e4m3 integers: every sum is exact in FP32
        Y = torch.from_numpy(v.astype(np.float32)).to(torch.float8_e4m3fn).view(torch.uint8).numpy()
    gate = g.integers(0, bins + 1, T).astype(np.uint8)  # bins itself: in no set
    plan = corr.Plan(S, N, T, precision=P, x_split=x_split)
    assert plan.splits == x_split
    acc = torch.full((bins, plan.acc_bytes // 4), 3, dtype=torch.int32 if prec == "int8" else torch.float32, device="cuda")
    plan.xengine_gated(pack_input(plan, Y), torch.from_numpy(gate).cuda(), bins, acc)
    acc = acc.cpu().numpy()
    y = torch.from_numpy(v).cuda().double().permute(2, 0, 1, 3)  # [C][S][T][2]
    r, q = y[..., 0].contiguous(), y[..., 1].contiguous()
    j, i = np.tril_indices(S)
    for b in range(bins):
        on = torch.from_numpy(gate == b).cuda()
        rt, qt = ((z * on).transpose(1, 2).contiguous() for z in (r, q))
        re, im = torch.bmm(r, rt) + torch.bmm(q, qt), torch.bmm(q, rt) - torch.bmm(r, qt)  # y_i conj(y_j)
        want = torch.stack([re[:, i, j], im[:, i, j]], -1).cpu().numpy() + 3 * x_split
        assert np.array_equal(acc_sum(acc[b], plan), want), b
