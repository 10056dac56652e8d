"""Training gradient of the learned flagger at the edges of its kernels' work
split: tile lists of one tile (fewer partial sums than the reduction has
slices), of a whole number of slices, and with a remainder; repeated tiles; and
tiles on every edge of the power array.  Against the FP64 oracle with the
bounds of test_gpu_cnn.py (FP32 sums of at most 2304 terms per activation and
512 pixels per partial: relative errors below 1e-5 of the largest gradient of a
layer, 1e-4 with margin)."""
import numpy as np
import pytest

import oracle
import paper_0910_1517_amd as corr
import synth
from test_gpu_cnn import dev, he_params, oracle_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [[0], [3, 3], [7, 0, 5], [1, 2, 4, 6, 7]])
def test_gradient_at_tile_counts(tiles):
    import torch
    S, T, C = 2, 128, 512
    power = synth.power_spectra(S, T, C, seed=21)
    labels = oracle.mad_tile_flags(power.astype(np.float64), 3.0)
    params = he_params(7, scale=0.7)
    ids = np.array(tiles, dtype=np.int32)
    cnn = corr.CNN(max_tiles=len(tiles))
    grads, losses = [], []
    for _ in range(2):
        loss = torch.full((1,), float("nan"), device="cuda")
        grad = torch.full((corr.CNN_PARAMS,), float("nan"), device="cuda")
        cnn.loss_grad(dev(params), dev(power), dev(labels), dev(ids), loss, grad)
        grads.append(grad.cpu().numpy())
        losses.append(loss.item())
    cnn.check_device_errors()
    assert np.array_equal(grads[0], grads[1]) and losses[0] == losses[1]  # fixed order of every sum
    x, y = oracle_inputs(power, ids, labels)
    loss64, g64 = oracle.cnn_loss_and_grad(params.astype(np.float64), x, y)
    assert abs(losses[0] - loss64) <= 1e-5 * loss64
    for lo, hi in [(0, 144), (144, 160), (160, 2464), (2464, 2480), (2480, 2624), (2624, 2625)]:
        assert np.abs(grads[0][lo:hi] - g64[lo:hi]).max() <= 1e-4 * np.abs(g64[lo:hi]).max(), (lo, hi)
