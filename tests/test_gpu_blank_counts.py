"""Voltage blanker with exact numbers of blanked samples per block, around the edges of its
replacement: less and more than a wave's lanes, whole and broken groups of loads in flight,
and the capacity of a wave's queue.  Bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_blank import gpu_table, run_blank

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("in_place", [True, False])
@pytest.mark.parametrize("block", [4096, 8192, 12288, 16384, 24576, 32768, 65536])
def test_counts(block, in_place):
    counts = [0, 1, 63, 64, 65, 255, 256, 257, 319, 320, 321, 1023, 1024, 1025] + (
        [2047, 2048, 2049, 3000] if block > 8192 else [block // 4 - 1, block // 4, block // 4 + 1, 1900])
    g = synth.rng(block, 72)
    x = np.empty((1, len(counts) * block), np.int8)
    for b, k in enumerate(counts):
        v = np.where(np.arange(block) % 2, 4, -4) + g.integers(-1, 2, block)  # median near 0, MAD 4
        where = g.choice(max(k, block // 4) if b % 2 else block, k, replace=False)
        v[where] = g.choice([-90, 90], k)
        x[0, b * block:(b + 1) * block] = v
    table, ref_table = gpu_table(5, 1, 1 << 12), oracle.blank_noise_table(5, 1, 1 << 12)
    out, _, cnt, st = run_blank(x, block, 3.0, table, sample0=3, in_place=in_place, pad=16)
    ref, rcnt, rst = oracle.mad_blank(x, block, 3.0, ref_table, sample0=3)
    assert rcnt[0].tolist() == counts
    assert np.array_equal(cnt, rcnt) and np.array_equal(st, rst)
    assert np.array_equal(out, ref)


@pytest.mark.parametrize("in_place", [True, False])
def test_no_value_is_kept(in_place):
    """A median between two values and a threshold below half a step: every sample is blanked."""
    x = np.tile(np.array([0, 1], np.int8), 16 * 33)[None]
    table, ref_table = gpu_table(5, 1, 1 << 6), oracle.blank_noise_table(5, 1, 1 << 6)
    out, _, cnt, _ = run_blank(x, 16, 0.5, table, sample0=0, in_place=in_place, pad=16)
    ref, rcnt, _ = oracle.mad_blank(x, 16, 0.5, ref_table, sample0=0)
    assert np.all(rcnt == 16) and np.array_equal(cnt, rcnt)
    assert np.array_equal(out, ref)
