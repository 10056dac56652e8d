"""The four-step F-engine's power cells leave through LDS in channel order: every
cell of every slot, at an address aligned to one cell only, and nothing beside them."""
import numpy as np
import pytest

import paper_0910_1517_amd as corr
import synth
from gpu_util import geom_dev, row_stride_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("half", [0, 1])
@pytest.mark.parametrize("prec", [corr.FP32, corr.INT8, corr.FP8_E4M3])
@pytest.mark.parametrize("N,T", [(512, 32), (512, 416), (2048, 32), (2048, 96), (4096, 32), (4096, 160)])
def test_cells_are_the_spectra_squared(N, T, prec, half):
    import torch
    S, C = 3, N // 2
    g = geom_dev(synth.make_geometry(2, seed=N).subset(np.arange(S)))
    rs = row_stride_for(N, T, 16)
    gen = torch.Generator(device="cuda").manual_seed(N + T)
    x = torch.randint(-127, 128, (S, rs), generator=gen, device="cuda", dtype=torch.int8)

    plan = corr.Plan(S, N, T, precision=corr.FP32)
    spec = plan.alloc("spectra", zero=False)
    plan.fengine(x, g, spec, None, row_stride=rs, spectrum0=3)
    y = spec.view(torch.float32).view(T // 2, C // 8, S, 8, 2, 2)  # [g][k/8][s][k%8][t%2][re im]
    want = (y.double() ** 2).sum(-1).permute(2, 0, 4, 1, 3).reshape(S, T, C)

    plan = corr.Plan(S, N, T, precision=prec, power_fp16=half)
    scale = torch.full((S, C), 30.0, device="cuda") if prec != corr.FP32 else None
    pad = torch.full((S * T * C + 2,), -1.0, device="cuda", dtype=torch.float16 if half else torch.float32)
    plan.fengine(x, g, plan.alloc("spectra", zero=False), scale, power=pad[1:-1], row_stride=rs, spectrum0=3)
    assert pad[0] == -1 and pad[-1] == -1
    got = pad[1:-1].view(S, T, C).double()
    # |Y|^2 of the phased FP32 spectra against |X|^2: two rotations and the two squares, a
    # few 2^-24 each; FP16 cells round |X|^2 / N^2 to 2^-11, or to 2^-25 below 2^-14
    if half:
        want = want / N ** 2
        assert ((got - want).abs() <= want * (2.0 ** -11 + 2e-6) + 2.0 ** -25).all()
    else:
        assert ((got - want).abs() <= want * 2e-6).all()


@pytest.mark.parametrize("S,T", [(1, 32), (3, 160), (5, 2080)])
def test_512_channel_fp32_spectra_with_and_without_cells(S, T):
    """FP32 spectra of 512 channels come from the four-step kernel without power cells
    and from the LDS-radix one with them: the same spectra, but for FP32 rounding."""
    import torch
    N = 1024
    geo = synth.make_geometry(3, seed=T).subset(np.arange(S))
    rs = row_stride_for(N, T, 16)
    gen = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randint(-127, 128, (S, rs), generator=gen, device="cuda", dtype=torch.int8)
    plan = corr.Plan(S, N, T, precision=corr.FP32)
    a, b = (plan.alloc("spectra", zero=False).fill_(fill) for fill in (7.0, 9.0))
    plan.fengine(x, geom_dev(geo), a, None, row_stride=rs, spectrum0=11)
    plan.fengine(x, geom_dev(geo), b, None, power=plan.alloc("power", zero=False), row_stride=rs, spectrum0=11)
    a, b = a.view(torch.float32).double(), b.view(torch.float32).double()
    # each kernel's error is near 1.5e-7 of the spectra's rms (FP32 sums of 10 stages);
    # the largest of some 1e6 differences stays within 9 times the two together
    assert (a - b).abs().max() <= 2e-6 * (a ** 2).mean().sqrt()


@pytest.mark.parametrize("lut", [0, 1])
@pytest.mark.parametrize("prec", [corr.FP32, corr.INT8, corr.FP8_E4M3])
@pytest.mark.parametrize("N", [512, 1024, 4096, 8192, 16384])
def test_spectra_do_not_depend_on_the_cells(N, prec, lut):
    """Launches with and without cells are separate kernels; their spectra are the
    same bytes (but for 512-channel FP32 spectra without the table, above), and the
    FP16 cells are the FP32 ones rounded."""
    import torch
    S, T = 3, 96
    g = geom_dev(synth.make_geometry(2, seed=N).subset(np.arange(S)))
    rs = row_stride_for(N, T, 16)
    gen = torch.Generator(device="cuda").manual_seed(N)
    x = torch.randint(-127, 128, (S, rs), generator=gen, device="cuda", dtype=torch.int8)
    scale = torch.full((S, N // 2), 30.0, device="cuda") if prec != corr.FP32 else None

    def run(cells, half):
        plan = corr.Plan(S, N, T, precision=prec, phase_lut=lut, power_fp16=half)
        spec = plan.alloc("spectra", zero=False).fill_(0xA5)
        power = plan.alloc("power", zero=False) if cells else None
        plan.fengine(x, g, spec, scale, power=power, row_stride=rs, spectrum0=1)
        return spec, power

    plain, _ = run(False, 0)
    full, p32 = run(True, 0)
    again, p16 = run(True, 1)
    assert torch.equal(full, again)
    if not (N == 1024 and prec == corr.FP32 and lut == 0):
        assert torch.equal(plain, full)
    assert torch.equal(p16, (p32 * 2.0 ** -(2 * (N.bit_length() - 1))).half())
