"""The Megopolis loop by windows: ancestors against the oracle (exact integers)
for numbers of steps around a group of five and each form's round (5, 10 and 20
steps), where the last, partial round begins; whole and prepared calls of one,
two and four particles per thread, both segment widths, and every batch shape."""
import numpy as np
import pytest

import oracle
from paper_2109_13504_amd import inputs

pytestmark = pytest.mark.gpu
STEPS = (1, 4, 5, 6, 9, 10, 11, 14, 15, 16, 19, 20, 21, 24, 26, 39, 40, 41, 354)


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2109_13504_amd import mgp
    return torch, torch.device("cuda:0"), mgp


@pytest.mark.parametrize("segment", [32, 64])
@pytest.mark.parametrize("n", [70001, 200003, 300007, 1 << 19])
def test_single(env, n, segment):
    torch, dev, mgp = env
    w = inputs.gaussian_weights(n, 2.0, 5)
    wd = torch.from_numpy(w).to(dev)
    idx = np.unique(np.concatenate([np.arange(70), np.arange(n - 70, n), np.arange(0, n, 997)])).astype(np.int32)
    r = mgp.Resampler(n)
    for B in STEPS:
        ref = oracle.resample_subset(w, "megopolis", B, 21, idx, stream_id=4, segment=segment)
        got = r.resample(wd, "megopolis", B=B, seed=21, stream_id=4, segment=segment).cpu().numpy()
        np.testing.assert_array_equal(got[idx], ref, err_msg=f"B={B}")
        r.compute_B(wd, "megopolis", B=B, seed=21, stream_id=4, segment=segment)
        got = r.resample_prepared(wd, "megopolis", B=B, seed=21, stream_id=4, segment=segment).cpu().numpy()
        np.testing.assert_array_equal(got[idx], ref, err_msg=f"prepared, B={B}")


@pytest.mark.parametrize("schedule", [1, 2])
@pytest.mark.parametrize("bt,ppt", [(64, 4), (64, 8), (128, 2), (128, 4), (128, 8), (256, 1), (256, 2), (256, 4)])
def test_batch(env, bt, ppt, schedule):
    torch, dev, mgp = env
    filters, refs = [], []
    for f, B in enumerate(STEPS):
        n = 900 + 331 * f
        w = inputs.gaussian_weights(n, 1.0, f)
        filters.append({"w": torch.from_numpy(w).to(dev), "anc": torch.zeros(n, dtype=torch.int32, device=dev), "B": B,
                        "seed": 9, "stream_id": f})
        refs.append(oracle.resample(w, "megopolis", B, 9, stream_id=f))
    plan = mgp.BatchPlan(filters, "megopolis", block_threads=bt, particles_per_thread=ppt, schedule=schedule)
    plan.run()
    torch.cuda.synchronize()
    for f, ref in zip(filters, refs):
        np.testing.assert_array_equal(f["anc"].cpu().numpy(), ref, err_msg=f"B={f['B']}")
    plan.close()
