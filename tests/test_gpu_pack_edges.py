"""Corner turn and requantisation at the edges of their work split: signal
counts that leave waves of a workgroup without a signal, the smallest and odd
spectrum counts, the smallest channel count, and buffers aligned to no more
than the calls ask for.  All bytes are exact."""
import numpy as np
import pytest

import paper_0910_1517_amd as corr
import synth

pytestmark = pytest.mark.gpu

PRECS = {"fp32": corr.FP32, "int8": corr.INT8, "e4m3": corr.FP8_E4M3}


@pytest.mark.parametrize("prec", sorted(PRECS))
@pytest.mark.parametrize("S,N,T", [(1, 512, 32), (3, 512, 96), (5, 2048, 32), (64, 512, 64), (30, 1024, 160)])
def test_xpack_layout(prec, S, N, T):
    import torch
    plan = corr.Plan(S, N, T, precision=PRECS[prec])
    g = synth.rng(S * N + T, 41)
    if prec == "fp32":
        a = g.standard_normal((S, T, N // 2, 2)).astype(np.float32)
    else:
        a = g.integers(0, 256, (S, T, N // 2, 2), dtype=np.uint8)
    spec = plan.alloc("spectra")
    plan.xpack(torch.from_numpy(a).cuda(), spec)
    got = corr.unpack_spectra(spec, PRECS[prec], S, N // 2, T)
    assert np.array_equal(got.view(np.uint8), a.view(np.uint8))


@pytest.mark.parametrize("prec", ["int8", "e4m3"])
@pytest.mark.parametrize("S,N,T", [(1, 512, 32), (3, 2048, 96)])
def test_requantize_same_codes_at_any_alignment(prec, S, N, T):
    import torch
    plan = corr.Plan(S, N, T, precision=PRECS[prec])
    g = synth.rng(S * N + T, 42)
    n = S * T * (N // 2) * 2
    a = torch.from_numpy((g.standard_normal(n) * 90).astype(np.float32)).cuda()
    a[:8] = torch.tensor([float("nan"), float("inf"), -float("inf"), 0.0, -0.0, 1e30, -1e30, 1e-30])
    scale = torch.from_numpy(g.uniform(0.5, 2.0, S * N // 2).astype(np.float32)).cuda()
    dt = torch.int8 if prec == "int8" else torch.uint8
    want = torch.zeros(n, dtype=dt, device="cuda")
    plan.requantize(a, scale, want)
    for off_in, off_scale, off_out in [(2, 0, 0), (0, 1, 0), (0, 0, 2), (2, 1, 6)]:
        src = torch.zeros(n + 8, device="cuda")[off_in:off_in + n].copy_(a)
        sc = torch.zeros(scale.numel() + 4, device="cuda")[off_scale:off_scale + scale.numel()].copy_(scale)
        dst = torch.zeros(n + 8, dtype=dt, device="cuda")[off_out:off_out + n]
        plan.requantize(src, sc, dst)
        assert torch.equal(dst, want), (off_in, off_scale, off_out)
