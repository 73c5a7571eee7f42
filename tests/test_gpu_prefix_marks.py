"""Systematic resampling at the edges of its search: blocks of 1792 outputs,
whose first groups the scan leaves, and inputs that mark their first output.
Every ancestor against the oracle (exact integers): whole and ragged last
blocks, on either side of the one-level tree (32768 inputs) and of the chunk
counts per block, weights that give one input nearly every output, and zeros
before, between and after the weights."""
import numpy as np
import pytest

import oracle
from paper_2109_13504_amd import inputs

pytestmark = pytest.mark.gpu
OUT = 1792  # outputs per block


def _check(w, seed):
    import torch

    from paper_2109_13504_amd import mgp
    r = mgp.PrefixResampler(len(w))
    got = r.resample(torch.from_numpy(w).cuda(), "systematic", seed=seed, stream_id=1).cpu().numpy()
    np.testing.assert_array_equal(got, oracle.resample_prefix(w, "systematic", seed, stream_id=1))


@pytest.mark.parametrize("n", [1, OUT - 1, OUT, OUT + 1, 18 * OUT, 19 * OUT - 1, 19 * OUT, 19 * OUT + 1, 64 * OUT,
                               (1 << 22) - 1, 1 << 22, (1 << 22) + 7, (1 << 24) + 1, (1 << 25) + 3])
def test_block_and_chunk_limits(n):
    _check(inputs.gaussian_weights(n, 1.0, n % 7), 11)


@pytest.mark.parametrize("n", [5000, 40000, 19 * OUT, 1000003])
def test_uneven_weights(n):
    g = np.random.Generator(np.random.PCG64(n))
    few = g.integers(0, n, 5)
    for lo, hi in ((0, n), (0, n // 3), (n // 2, n), (n // 3, n // 2)):
        w = np.zeros(n, np.float32)
        w[lo:hi] = g.random(hi - lo, dtype=np.float32)
        _check(w, 3)  # zeros at the ends
        w[few] = 1e9  # and a few inputs with nearly every output
        _check(w, 4)
    w = np.zeros(n, np.float32)
    for k in (0, n // 2, n - 1):  # one input only
        w[:] = 0.0
        w[k] = 3.0
        _check(w, 5)
    _check(np.ones(n, np.float32), 6)  # one output each: the thresholds meet the sums' spacing
