"""A prepared loop after a whole resample: it sees the weights of that call, also
where the call's own loop read them in place and they have changed since, and
where its outputs lie over them. Ancestors against the oracle (exact integers:
no tolerance), one size per form of the loop and of the launches before it."""
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


def _weights(torch, dev, n, shift, seed):
    w = inputs.gaussian_weights(n, 2.0, seed)
    wd = torch.zeros(n + 64, device=dev)[shift:shift + n]
    wd.copy_(torch.from_numpy(w))
    return w, wd


# the split loop, one, two and four particles per thread, the finalize step in a launch of its own
@pytest.mark.parametrize("n", [32769, 65536, 70001, 131072, 200003, 600011, (1 << 20) + 13, (1 << 21) + 5, 1 << 22])
@pytest.mark.parametrize("shift", [0, 1])
def test_weights_changed_since(env, n, shift):
    torch, dev, mgp = env
    B, seed = 13, 5
    w, wd = _weights(torch, dev, n, shift, n % 13)
    ref = oracle.resample(w, "megopolis", B, seed)
    r = mgp.Resampler(n)
    np.testing.assert_array_equal(r.resample(wd, "megopolis", B=B, seed=seed).cpu().numpy(), ref)
    wd.fill_(1.0)
    np.testing.assert_array_equal(r.resample_prepared(wd, "megopolis", B=B, seed=seed).cpu().numpy(), ref)
    # another buffer, and the ancestors over the weights
    other = torch.rand(n, device=dev)
    np.testing.assert_array_equal(r.resample_prepared(other, "megopolis", B=B, seed=seed).cpu().numpy(), ref)
    wd.copy_(torch.from_numpy(w))
    r.resample(wd, "megopolis", B=B, seed=seed)
    over = r.resample_prepared(wd, "megopolis", B=B, seed=seed, out=wd.view(torch.int32))
    np.testing.assert_array_equal(over.cpu().numpy(), ref)


@pytest.mark.parametrize("n", [70001, 600011, (1 << 20) + 13])
def test_fused_copy(env, n):
    torch, dev, mgp = env
    d, B, seed = 4, 9, 7
    w, wd = _weights(torch, dev, n, 0, 3)
    states = torch.randn((n, d), device=dev)
    ref = oracle.resample(w, "megopolis", B, seed)
    rows = states.cpu().numpy()[ref]
    r = mgp.Resampler(n)
    out, anc = r.resample_gather(wd, states, "megopolis", B=B, seed=seed)
    np.testing.assert_array_equal(anc.cpu().numpy(), ref)
    wd.fill_(float("nan"))
    out, anc = r.resample_gather_prepared(wd, states, "megopolis", B=B, seed=seed)
    np.testing.assert_array_equal(anc.cpu().numpy(), ref)
    np.testing.assert_array_equal(out.cpu().numpy(), rows)


@pytest.mark.parametrize("n", [100, 1023, 1024, 1025, 5000, 70001, 200003])
def test_after_m_outputs(env, n):
    """mgp_resample_m leaves the workspace prepared at every size, whatever M."""
    torch, dev, mgp = env
    B, seed = 11, 3
    r = mgp.Resampler(n)
    for m in (1, n // 2, n, n + 777):
        w, wd = _weights(torch, dev, n, 0, m % 17)
        ref = oracle.resample(w, "megopolis", B, seed)
        got = r.resample_m(wd, m, "megopolis", B=B, seed=seed)
        np.testing.assert_array_equal(got.cpu().numpy(), oracle.resample_m(w, m, "megopolis", B, seed))
        wd.fill_(2.0)
        np.testing.assert_array_equal(r.resample_prepared(wd, "megopolis", B=B, seed=seed).cpu().numpy(), ref,
                                      err_msg=f"m={m}")


@pytest.mark.parametrize("n", [5000, 20001, 32768])
def test_small_calls_leave_nothing(env, n):
    torch, dev, mgp = env
    _, wd = _weights(torch, dev, n, 0, 1)
    r = mgp.Resampler(n)
    r.resample(wd, "megopolis", B=8, seed=2)
    assert (r.resample_prepared(wd, "megopolis", B=8, seed=2) == -1).all()
