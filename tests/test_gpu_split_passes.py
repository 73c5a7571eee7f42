"""The split Megopolis loop: ancestors against the oracle (exact) for numbers of
steps around a u block (5), a pass (30) and two passes, where its producers
and its chains change buffers, with the weights in LDS (n <= 8192) and in
global memory, prepared and in one call, with whole and ragged blocks of 64
particles and both segment widths."""
import numpy as np
import pytest

import oracle
from paper_2109_13504_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [7, 64, 1000, 8192, 8193, 20000, 65536])
def test_steps(n):
    import torch

    from paper_2109_13504_amd import mgp
    w = inputs.gaussian_weights(n, 2.0, 5)
    wd = torch.from_numpy(w).cuda()
    idx = np.unique(np.concatenate([np.arange(min(n, 130)), np.arange(max(0, n - 130), n)])).astype(np.int32)
    r = mgp.Resampler(n)
    for B in (1, 4, 5, 6, 10, 11, 25, 29, 30, 31, 34, 36, 45, 59, 60, 61, 89, 90, 91, 121, 354):
        ref = oracle.resample_subset(w, "megopolis", B, 21, idx, stream_id=4)
        got = r.resample(wd, "megopolis", B=B, seed=21, stream_id=4).cpu().numpy()
        np.testing.assert_array_equal(got[idx], ref, err_msg=f"B={B}")
        r.compute_B(wd, "megopolis", B=B, seed=21, stream_id=4)
        got = r.resample_prepared(wd, "megopolis", B=B, seed=21, stream_id=4).cpu().numpy()
        np.testing.assert_array_equal(got[idx], ref, err_msg=f"prepared, B={B}")


@pytest.mark.parametrize("segment", [32, 64])
@pytest.mark.parametrize("n", [5000, 30001])
def test_segments(n, segment):
    import torch

    from paper_2109_13504_amd import mgp
    w = inputs.gaussian_weights(n, 1.0, 6)
    idx = np.arange(0, n, 13).astype(np.int32)
    got = mgp.resample(torch.from_numpy(w).cuda(), B=37, seed=8, stream_id=1, segment=segment)[0].cpu().numpy()
    np.testing.assert_array_equal(got[idx], oracle.resample_subset(w, "megopolis", 37, 8, idx, stream_id=1,
                                                                   segment=segment))
