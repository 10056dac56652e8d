"""Corner turn of so many FP32 spectra that the launch extent matters: 2^31 cells a
signal (2^30 chunks), for the signal counts that leave waves of a workgroup without a
signal.  A launch has fewer than 2^32 threads in x."""
import pytest

import paper_0910_1517_amd as corr

pytestmark = [pytest.mark.gpu, pytest.mark.slow]


@pytest.mark.parametrize("S", [1, 3])
def test_fp32_cells_of_a_signal_2_31(S):
    import torch
    N, T = 16384, 1 << 18
    C = N // 2
    plan = corr.Plan(S, N, T, precision=corr.FP32)
    gen = torch.Generator(device="cuda").manual_seed(S)
    cells = torch.empty(S, T, C, dtype=torch.int64, device="cuda")  # one complex64 each
    for part in cells.view(-1).split(1 << 28):
        part.random_(generator=gen)
    spec = torch.zeros(plan.spectra_bytes, dtype=torch.uint8, device="cuda")
    plan.xpack(cells.view(torch.float32), spec)
    got = spec.view(torch.int64).view(T // 2, C // 8, S, 8, 2)
    step = 1 << 13
    for s in range(S):
        for g in range(0, T // 2, step):
            want = cells[s, 2 * g:2 * (g + step)].view(step, 2, C // 8, 8)
            assert torch.equal(got[g:g + step, :, s].permute(0, 3, 1, 2), want), (s, g)
    del cells, spec, got, want, part
    torch.cuda.empty_cache()
