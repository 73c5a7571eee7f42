"""mgp_server_copy_outputs by one kernel: the words are those of the request's
outputs at sizes around the kernel's chunk (2048 words), whole and ragged, for
destinations with and without 16-byte alignment, nothing beside them is
written, a destination in host memory still takes the runtime's copy, and the
copy can be captured and replayed."""
import numpy as np
import pytest

from paper_2109_13504_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d", [(1, 1), (2047, 3), (2048, 4), (2049, 4), (4096, 8), (131075, 5)])
def test_copied_words(n, d):
    import torch

    from paper_2109_13504_amd import mgp
    w_np, st_np = inputs.gaussian_weights_and_states(n, 1.0, d, 7)
    w, st = torch.from_numpy(w_np).cuda(), torch.from_numpy(st_np).cuda()
    k_ref = mgp.resample(w, seed=31, stream_id=2)[0].cpu().numpy()
    x_ref = st_np.reshape(n, d)[k_ref]
    srv = mgp.Server("megopolis", d=d, hbm_budget=1 << 26, streams=1, max_batch=1, max_n=1 << 18)
    try:
        t = srv.submit(w, seed=31, stream_id=2, states=st)
        assert srv.wait(t, 60000.0)["state"] == 2
        for dev, off in (("cuda", 0), ("cuda", 1), ("cuda", 3), ("cpu", 0)):
            anc = torch.full((n + 8,), -7, dtype=torch.int32, device=dev)
            out = torch.full((n * d + 8,), -7.0, dtype=torch.float32, device=dev)
            if dev == "cpu":
                anc, out = anc.pin_memory(), out.pin_memory()
            mgp.mgp_server_copy_outputs(srv.handle, t, anc.data_ptr() + 4 * off, out.data_ptr() + 4 * off,
                                        mgp.current_stream())
            torch.cuda.synchronize()
            a, x = anc.cpu().numpy(), out.cpu().numpy()
            np.testing.assert_array_equal(a[off:off + n], k_ref)
            np.testing.assert_array_equal(x[off:off + n * d].reshape(n, d), x_ref)
            assert (a[:off] == -7).all() and (a[off + n:] == -7).all()
            assert (x[:off] == -7).all() and (x[off + n * d:] == -7).all()
        anc = torch.zeros(n, dtype=torch.int32, device="cuda")
        out = torch.zeros(n * d, dtype=torch.float32, device="cuda")
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, capture_error_mode="thread_local"):
            mgp.mgp_server_copy_outputs(srv.handle, t, anc.data_ptr(), out.data_ptr(),
                                        torch.cuda.current_stream().cuda_stream)
        for _ in range(3):
            anc.zero_()
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            np.testing.assert_array_equal(anc.cpu().numpy(), k_ref)
            np.testing.assert_array_equal(out.cpu().numpy().reshape(n, d), x_ref)
        srv.release(t)
    finally:
        srv.close()
