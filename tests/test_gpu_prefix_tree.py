"""The prefix-sum resamplers' tree of group sums: every ancestor against the
oracle (exact integers) where the number of levels, the passes per block, the
place of the finalize step or the systematic search change, and for weights
over fp32's whole range."""
import numpy as np
import pytest

import oracle
from paper_2109_13504_amd import inputs, mgp as _  # noqa: F401

pytestmark = pytest.mark.gpu
METHODS = ["multinomial", "systematic"]


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2109_13504_amd import mgp
    return torch, torch.device("cuda:0"), mgp


def _check(env, w, method, seed=5, shift=0):
    torch, dev, mgp = env
    n = len(w)
    base = torch.zeros(n + 4, device=dev)
    wd = base[shift:shift + n]
    wd.copy_(torch.from_numpy(w))
    r = mgp.PrefixResampler(n)
    got = r.resample(wd, method, seed=seed, stream_id=3).cpu().numpy()
    np.testing.assert_array_equal(got, oracle.resample_prefix(w, method, seed, stream_id=3))
    return r.last_stats()


@pytest.mark.parametrize("method", METHODS)
@pytest.mark.parametrize("n", [15, 16, 17, 255, 1023, 1024, 1025, 32752, 32768, 32769, 32785, (1 << 19) - 1, 1 << 19,
                               524305, (1 << 21), (1 << 21) + 1])
def test_level_and_pass_limits(env, method, n):
    w = inputs.gaussian_weights(n, 3.0, n % 11)
    st = _check(env, w, method)
    s = float(np.sum(w.astype(np.float64)))
    # n additions in fp64, each rounded once
    assert abs(st["w_sum"] - s) <= n * 2.0**-52 * s
    _check(env, w, method, shift=1)


@pytest.mark.parametrize("method", METHODS)
def test_sorted_and_sparse_weights(env, method):
    """Long runs of tiny or zero weights: one block's outputs then span more
    inputs than it adds up in tiles, from just below that limit to far above."""
    n = 300007
    w = np.sort(inputs.gaussian_weights(n, 4.0, 1))
    _check(env, w, method)
    _check(env, w[::-1].copy(), method)
    for gap in (16000, 16368, 16384, 16400, 40000):
        w = np.zeros(n, np.float32)
        w[::gap] = 1.0
        w[-1] = 2.0
        _check(env, w, method)


@pytest.mark.parametrize("method", METHODS)
@pytest.mark.parametrize("scale", [1e-38, 1e-44, 3e38, 1.0])
def test_fp32_range(env, method, scale):
    """Subnormal and huge weights, negative zeros, weights below the fixed
    point's resolution beside large ones."""
    n = 70001
    g = np.random.Generator(np.random.PCG64(3))
    w = (g.random(n) * scale).astype(np.float32)
    w[::7] = -0.0
    w[::13] = np.float32(1e-45)
    w[n // 2] = np.float32(scale)
    _check(env, w, method)
