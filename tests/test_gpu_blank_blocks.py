"""Voltage blanker at the edges of its kernels' block sizes: the largest block of
each, one chunk more, and blocks that fill the last one badly, in place and out
of place, with a ragged last block; and data that put the median between two
values.  Bit-exact against the oracle, like test_gpu_blank.py."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_blank import data, gpu_table, run_blank

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("in_place", [True, False])
@pytest.mark.parametrize("kind", ["heavy", "low", "bits4"])
@pytest.mark.parametrize("block", [16, 2032, 2048, 2064, 4096, 4112, 8192, 8208, 12288, 12304, 16384, 16400, 20000,
                                   24576, 24592, 32768, 32784, 65536])
def test_block_sizes(block, kind, in_place):
    S, n = 2, 2 * block + max(1, block // 3) + 5
    if kind == "bits4":  # four-bit samples: whole blocks of few values
        g = synth.rng(block, 71)
        x = np.clip(np.rint(g.normal(0.3, 1.5, (S, n))), -8, 7).astype(np.int8)
        x[:, :block] = np.where(np.arange(block) % 2, 3, -2)  # median 0.5 (or one of the two), MAD 2.5 or 0
    else:
        x = data(kind, S, n, seed=block)
    table = gpu_table(5, S, 1 << 12)
    ref_table = oracle.blank_noise_table(5, S, 1 << 12)
    for M in (3.0, 0.25):  # 0.25: most samples of a block are blanked
        out, tail, cnt, st = run_blank(x, block, M, table, sample0=3, in_place=in_place, pad=16)
        ref, rcnt, rst = oracle.mad_blank(x, block, M, ref_table, sample0=3)
        assert np.array_equal(st, rst)
        assert np.array_equal(cnt, rcnt)
        assert np.array_equal(out, ref)
        assert np.all(tail == (0x5A if in_place else 0x33))
