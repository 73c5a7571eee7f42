"""The prefix-sum resamplers on weights that make a block's outputs span much of
the input (long runs of tiny weights beside a few large ones), and at addresses
of every alignment: ancestors against the oracle (exact integers) at sizes of
each number of tree levels and on both sides of the sizes where the scan moves
and where unaligned weights are copied."""
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


def _check(env, w, method, shift=0, seed=9):
    torch, dev, mgp = env
    n = len(w)
    wd = torch.zeros(n + 64, device=dev)[shift:shift + n]
    wd.copy_(torch.from_numpy(w))
    got = mgp.PrefixResampler(n).resample(wd, method, seed=seed, stream_id=2).cpu().numpy()
    np.testing.assert_array_equal(got, oracle.resample_prefix(w, method, seed, stream_id=2))


# two, three and four levels of the tree; whole and ragged last groups and blocks
@pytest.mark.parametrize("n", [32769, 60000, 524288, 524289, 1 << 20, 8388609, (1 << 24) + 5])
@pytest.mark.parametrize("kind", ["rising", "falling", "few"])
def test_systematic_long_runs(env, n, kind):
    w = inputs.gaussian_weights(n, 4.0, n % 5)
    if kind == "few":  # three groups hold nearly every output: long runs of starts and searches
        w = (w * 1e-4).astype(np.float32)
        w[[5, n // 2, n - 3]] = 1e5
    else:
        w = np.sort(w) if kind == "rising" else np.sort(w)[::-1].copy()
    _check(env, w, "systematic", shift=n % 3)


@pytest.mark.parametrize("method", ["multinomial", "systematic"])
@pytest.mark.parametrize("n", [17, 5003, 40001, (1 << 21) - 1, 1 << 21, (1 << 21) + 3])
def test_alignments(env, method, n):
    w = inputs.gaussian_weights(n, 2.0, n % 7)
    for shift in (0, 1, 2, 3, 4, 8, 16):
        _check(env, w, method, shift=shift, seed=20 + shift)
