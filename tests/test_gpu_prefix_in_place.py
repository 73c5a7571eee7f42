"""The prefix-sum resamplers with outputs over the weights: the search reads the
weights while it writes ancestors, so these calls work on a copy. Ancestors
against the oracle (exact integers: no tolerance), for all of the weights, a
part of them, and the stats record among them, on each side of the sizes where
the scan, the number of chunks per block and the finalize step change place."""
import numpy as np
import pytest

import oracle
from paper_2109_13504_amd import inputs

pytestmark = pytest.mark.gpu
METHODS = ["multinomial", "systematic"]


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2109_13504_amd import mgp
    return torch, torch.device("cuda:0"), mgp


@pytest.mark.parametrize("method", METHODS)
@pytest.mark.parametrize("n", [1, 33, 5000, 32768, 32769, 100003, (1 << 22) + 13, (1 << 24) + 5])
def test_ancestors_over_the_weights(env, method, n):
    torch, dev, mgp = env
    w = inputs.gaussian_weights(n, 3.0, n % 7)
    ref = oracle.resample_prefix(w, method, 11, stream_id=2)
    r = mgp.PrefixResampler(n)
    for shift in (0, 1):  # 16-byte aligned weights, and not
        buf = torch.zeros(2 * n + 8, device=dev)
        wd = buf[shift:shift + n]
        wd.copy_(torch.from_numpy(w))
        got = r.resample(wd, method, seed=11, stream_id=2, out=wd.view(torch.int32))
        np.testing.assert_array_equal(got.cpu().numpy(), ref, err_msg=f"shift {shift}")
        # over the second half of the weights only
        wd.copy_(torch.from_numpy(w))
        part = buf[shift + n // 2:shift + n // 2 + n].view(torch.int32)
        got = r.resample(wd, method, seed=11, stream_id=2, out=part)
        np.testing.assert_array_equal(got.cpu().numpy(), ref, err_msg=f"shift {shift}, second half")


@pytest.mark.parametrize("method", METHODS)
def test_sparse_weights_and_stats_record(env, method):
    """Weights so sparse that the systematic search descends output by output;
    and the caller's stats record among the weights, which the first kernel
    after the reduction writes."""
    torch, dev, mgp = env
    n = 300008
    w = np.zeros(n, np.float32)
    w[::40000] = 1.0
    w[-1] = 2.0
    ref = oracle.resample_prefix(w, method, 5)
    r = mgp.PrefixResampler(n)
    wd = torch.from_numpy(w).to(dev)
    got = r.resample(wd, method, seed=5, out=wd.view(torch.int32))
    np.testing.assert_array_equal(got.cpu().numpy(), ref)

    w = inputs.gaussian_weights(n, 2.0, 3)
    ref = oracle.resample_prefix(w, method, 5)
    wd = torch.from_numpy(w).to(dev)
    anc = torch.zeros(n, dtype=torch.int32, device=dev)
    mgp.mgp_resample_prefix(wd.data_ptr(), n, mgp.PREFIX_METHODS[method], 5, 0, anc.data_ptr(), wd.data_ptr() + 4096,
                            r.workspace.data_ptr(), r.ws_bytes, mgp.current_stream())
    np.testing.assert_array_equal(anc.cpu().numpy(), ref)
    st = mgp.decode_stats(wd[1024:1024 + r.stats.numel() * r.stats.element_size() // 4].view(r.stats.dtype))
    assert st["status"] == 0 and st["n"] == n and st["w_max"] == np.float32(w.max())
