"""Gated X-engine over bin counts that fill its workgroups' pairs of bins and
that leave one empty, signal counts at the edges of its tiles, and gates that
leave bins without a spectrum: each bin's sums are the X-engine's over that
bin's spectra alone, exactly."""
import numpy as np
import pytest

import paper_0910_1517_amd as corr
import synth
from gpu_util import acc_sum, pack_input

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["int8", "e4m3"])
@pytest.mark.parametrize("S", [1, 9, 32, 33, 64])
@pytest.mark.parametrize("bins", [1, 2, 3, 4, 5])
def test_bins_equal_their_spectra_alone(S, bins, prec):
    import torch
    T, N = 96, 512
    P = {"int8": corr.INT8, "e4m3": corr.FP8_E4M3}[prec]
    g = synth.rng(100 * S + bins, 61)
    if prec == "int8":
        Y = g.integers(-127, 128, (S, T, N // 2, 2), dtype=np.int8)
    else:  # small e4m3 integers: every sum is exact in FP32
        Y = torch.from_numpy(g.integers(-4, 5, (S, T, N // 2, 2)).astype(np.float32)).to(torch.float8_e4m3fn)
        Y = Y.view(torch.uint8).numpy()
    gate = g.integers(0, bins + 1, T).astype(np.uint8)  # bins itself: in no set
    gate[gate == bins // 2] = bins  # and one bin without a spectrum
    plan = corr.Plan(S, N, T, precision=P, x_split=3)
    n = plan.acc_bytes // 4
    dt = torch.int32 if prec == "int8" else torch.float32
    acc = torch.zeros(bins, n, dtype=dt, device="cuda")
    plan.xengine_gated(pack_input(plan, Y), torch.from_numpy(gate).cuda(), bins, acc)
    for b in range(bins):
        alone = np.where((gate == b)[None, :, None, None], Y, np.zeros_like(Y))
        one = corr.Plan(S, N, T, precision=P, x_split=3)
        want = one.alloc("acc")
        one.xengine(pack_input(one, alone), want)
        torch.cuda.synchronize()
        assert np.array_equal(acc_sum(acc[b].cpu().numpy(), plan), acc_sum(want.cpu().numpy(), one)), b
