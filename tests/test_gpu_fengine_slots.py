"""The F-engines choose how many consecutive spectra a workgroup takes from the
size of the call.  A spectrum's arithmetic does not depend on that choice: a
short call's spectra and power cells are, bit for bit, the first ones of a long
call on the same rows."""
import numpy as np
import pytest

import paper_0910_1517_amd as corr
import synth
from gpu_util import geom_dev, row_stride_for

pytestmark = pytest.mark.gpu

PRECS = {"fp32": corr.FP32, "int8": corr.INT8, "e4m3": corr.FP8_E4M3}


@pytest.mark.parametrize("lut", [0, 1])
@pytest.mark.parametrize("prec", sorted(PRECS))
@pytest.mark.parametrize("N", [512, 1024, 2048, 4096, 8192, 16384])
def test_short_calls_equal_the_start_of_a_long_one(N, prec, lut):
    import torch
    S, long = 5, 16384 * 512 // N
    geo = synth.make_geometry(3, seed=N).subset(np.arange(S))
    g = geom_dev(geo)
    rs = row_stride_for(N, long, 16)
    gen = torch.Generator(device="cuda").manual_seed(N)
    x = torch.randint(-127, 128, (S, rs), generator=gen, device="cuda", dtype=torch.int8)
    scale = torch.rand(S, N // 2, generator=gen, device="cuda") * 40 + 20 if prec != "fp32" else None

    def spectra(T, cells):
        plan = corr.Plan(S, N, T, precision=PRECS[prec], phase_lut=lut, power_fp16=1)
        spec = plan.alloc("spectra", zero=False).fill_(0xA5)
        power = plan.alloc("power", zero=False).fill_(-1) if cells else None
        plan.fengine(x, g, spec, scale, power=power, row_stride=rs, spectrum0=7)
        return spec, power.view(S, T, N // 2) if cells else None

    for cells in (False, True):
        want, pw = spectra(long, cells)
        for T in (32, 96, 128, 416):
            got, pg = spectra(T, cells)
            assert torch.equal(got, want[:got.numel()]), T
            if cells:
                assert torch.equal(pg, pw[:, :T]), T
