"""FP32 X-engine over the exponents whose visibilities are normal FP32 numbers, and with one
signal at the smallest components that its three BF16 parts hold exactly: the bound of
test_gpu_x_fp32.py (products exact to 2^-24, sums of 16 spectra rounded at 2^-23), which
no product and no part below the normal numbers may break."""
import numpy as np
import pytest

import synth
from test_gpu_x_fp32 import reference, visibilities

pytestmark = pytest.mark.gpu


def check(Y):
    T = Y.shape[1]
    re, im = visibilities(Y, 1)
    V, scale = reference(Y)
    assert (np.abs(re + 1j * im - V) / scale).max() <= 2.0 ** -24 * (8 + T / 16)


@pytest.mark.parametrize("S", [9, 40])
@pytest.mark.parametrize("T", [32, 256])
def test_amplitudes(S, T):
    g = synth.rng(S + T, 95)
    Y = g.standard_normal((S, T, 256, 2)) + 0.5 * g.standard_normal((1, T, 256, 2))
    check(np.ldexp(Y, g.integers(-61, 56, (1, 1, 256, 1))).astype(np.float32))  # 4e-19 .. 4e16 a channel


@pytest.mark.parametrize("S", [9, 40])
def test_one_tiny_signal(S):
    T, g = 64, synth.rng(S, 96)
    Y = g.uniform(1, 2, (S, T, 256, 2)) * g.choice([-1.0, 1.0], (S, T, 256, 2))
    e = np.full(S, 40)
    e[S // 2] = -110
    Y = np.ldexp(Y, e[:, None, None, None]).astype(np.float32)
    re, im = visibilities(Y, 1)
    V, scale = reference(Y)
    j, i = np.tril_indices(S)
    normal = ~((i == S // 2) & (j == S // 2))  # its own power is 2^-214
    assert (np.abs(re + 1j * im - V) / scale)[:, normal].max() <= 2.0 ** -24 * (8 + T / 16)
