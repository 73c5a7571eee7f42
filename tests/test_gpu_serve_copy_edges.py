"""mgp_server_copy_outputs where its one kernel must not change what the two
copies before it did: destinations that overlap (the ancestors are copied first,
the states over them), and a thread whose last HIP call failed."""
import ctypes
import re

import numpy as np
import pytest

from paper_2109_13504_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def served():
    import torch

    from paper_2109_13504_amd import mgp
    n, d = 131075, 5
    w_np, st_np = inputs.gaussian_weights_and_states(n, 1.0, d, 7)
    w, st = torch.from_numpy(w_np).cuda(), torch.from_numpy(st_np).cuda()
    k_ref = mgp.resample(w, seed=31, stream_id=2)[0].cpu().numpy()
    srv = mgp.Server("megopolis", d=d, hbm_budget=1 << 26, streams=1, max_batch=1, max_n=1 << 18)
    t = srv.submit(w, seed=31, stream_id=2, states=st)
    assert srv.wait(t, 60000.0)["state"] == 2
    yield torch, mgp, srv, t, n, d, k_ref, st_np.reshape(n, d)[k_ref].reshape(-1)
    srv.release(t)
    srv.close()


@pytest.mark.parametrize("gap", [0, 1, 1000, 131074, -1, -4 * 131075])
def test_overlapping_destinations(served, gap):
    """The states' destination `gap` words after the ancestors'."""
    torch, mgp, srv, t, n, d, k_ref, x_ref = served
    buf = torch.zeros(3 * n * d, dtype=torch.int32, device="cuda")
    anc, out = n * d, n * d + gap
    want = np.zeros(buf.numel(), np.int32)
    want[anc:anc + n] = k_ref
    want[out:out + n * d] = x_ref.view(np.int32)
    mgp.mgp_server_copy_outputs(srv.handle, t, buf.data_ptr() + 4 * anc, buf.data_ptr() + 4 * out,
                                mgp.current_stream())
    np.testing.assert_array_equal(buf.cpu().numpy(), want)


def test_an_older_error_is_not_this_call(served):
    torch, mgp, srv, t, n, d, k_ref, x_ref = served
    anc = torch.zeros(n, dtype=torch.int32, device="cuda")
    out = torch.zeros(n * d, device="cuda")
    torch.cuda.synchronize()
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL(re.search(r"\S*/libamdhip64\.so\S*", f.read()).group(0))
    assert hip.hipSetDevice(4096) != 0  # refused, and remembered as the thread's last error
    try:
        mgp.mgp_server_copy_outputs(srv.handle, t, anc.data_ptr(), out.data_ptr(), mgp.current_stream())
    finally:
        hip.hipGetLastError()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(anc.cpu().numpy(), k_ref)
    np.testing.assert_array_equal(out.cpu().numpy(), x_ref)
