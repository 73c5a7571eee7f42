"""mgp_resample in two launches: the finalize step inside the accept loop, with
offsets drawn by the reduction before B is known.

Ancestors against the oracle and the stats against mgp_compute_B's, field by
field (both exact), on both sides of every size limit of the dispatch, with B
from epsilon, fixed, clamped and past the early offsets' limit."""
import numpy as np
import pytest

import oracle
from paper_2109_13504_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2109_13504_amd import mgp
    return torch, torch.device("cuda:0"), mgp


def _check(env, variant, n, w, b_max=0, **kw):
    torch, dev, mgp = env
    wd = torch.from_numpy(w).to(dev)
    r = mgp.Resampler(n, b_max=b_max)
    got = r.resample(wd, variant, seed=17, stream_id=2, **kw).cpu().numpy()
    st = r.last_stats()
    r.compute_B(wd, variant, seed=17, stream_id=2, **kw)
    assert st == r.last_stats()
    idx = np.unique(np.concatenate([np.arange(300), np.arange(n - 300, n), np.arange(0, n, n // 500 + 1)])).astype(np.int32)
    ref = oracle.resample_subset(w, variant, st["B"], 17, idx, stream_id=2)
    np.testing.assert_array_equal(got[idx], ref)
    return st


@pytest.mark.parametrize("variant,n", [("megopolis", 8193), ("megopolis", 1 << 16), ("megopolis", (1 << 16) + 1),
                                       ("megopolis", 1 << 17), ("megopolis", (1 << 17) + 1), ("megopolis", 1 << 18),
                                       ("megopolis", (1 << 18) + 1), ("megopolis", 1 << 20),
                                       ("megopolis", (1 << 20) + 1), ("metropolis", 4097), ("metropolis", 1 << 18),
                                       ("metropolis", (1 << 18) + 1), ("c1", 50001), ("c2", 1 << 18), ("c2", 4100)])
def test_sizes(env, variant, n):
    w = inputs.gaussian_weights(n, 2.0, 9)
    _check(env, variant, n, w, epsilon=0.01)
    for B in (1, 9, 10, 11, 21):
        _check(env, variant, n, w, B=B)


@pytest.mark.parametrize("n", [9000, 70000, 150000, 300000])
def test_many_offsets(env, n):
    """B beyond one block of early offsets (4096), clamped to b_max; and b_max
    past the early offsets' limit, which goes back to three launches."""
    w = np.full(n, np.float32(1e-30))
    w[17] = np.float32(1.0)
    st = _check(env, "megopolis", n, w, b_max=4099, epsilon=0.01)
    assert st["B"] == 4099 and st["clamped"] == 1
    w = inputs.gaussian_weights(n, 2.0, 4)
    _check(env, "megopolis", n, w, b_max=65537, epsilon=0.01)


@pytest.mark.parametrize("variant,n", [("megopolis", 20000), ("megopolis", 200000), ("c1", 20000)])
def test_invalid_and_replays(env, variant, n):
    """Invalid weights give -1 and the status; the same graph replayed with
    other weights in between gives each one's own result."""
    torch, dev, mgp = env
    w = inputs.gaussian_weights(n, 2.0, 1)
    other = inputs.gaussian_weights(n, 3.0, 2)
    wd = torch.from_numpy(w).to(dev)
    r = mgp.Resampler(n)
    out = torch.empty(n, dtype=torch.int32, device=dev)
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    r.resample(wd, variant, epsilon=0.01, seed=3, out=out)
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        r.resample(wd, variant, epsilon=0.01, seed=3, out=out)
    for x in (w, other, w):
        wd.copy_(torch.from_numpy(x))
        g.replay()
        torch.cuda.synchronize()
        B = r.last_stats()["B"]
        assert B == oracle.B_from_weights(x, 0.01)[0]
        idx = np.arange(0, n, 97, dtype=np.int32)
        np.testing.assert_array_equal(out.cpu().numpy()[idx], oracle.resample_subset(x, variant, B, 3, idx))
    wd[n // 2] = float("nan")
    assert (r.resample(wd, variant, epsilon=0.01, seed=3).cpu().numpy() == -1).all()
    assert r.last_stats()["status"] == mgp.MGP_EWEIGHTS
