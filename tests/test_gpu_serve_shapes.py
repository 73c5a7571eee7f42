"""The server's two launch shapes: micro-batches of up to 2^18 particles and
larger ones give the same ancestors and rows, the oracle's (exact)."""
import numpy as np
import pytest

import oracle
from paper_2109_13504_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[1], [300, 1], [1 << 18], [(1 << 18) + 1], [1 << 15] * 8, [(1 << 15) + 1] * 8,
                                   [5003, 257, 256, 255, 100003], [100003, 1 << 17, 70001]])
def test_around_the_limit(sizes):
    import torch

    from paper_2109_13504_amd import mgp
    d = 3
    srv = mgp.Server("megopolis", d=d, hbm_budget=1 << 28, streams=1, max_batch=8, max_batch_particles=1 << 21)
    try:
        held = []
        for f, n in enumerate(sizes):
            w, st = inputs.gaussian_weights_and_states(n, 2.0, d, f)
            wd, sd = torch.from_numpy(w).cuda(), torch.from_numpy(st.reshape(n, d)).cuda()
            held.append((srv.submit(wd, B=0 if f % 2 else 23, epsilon=0.01, seed=6, stream_id=f, states=sd), w, st, wd, sd))
        for f, (t, w, st, _, _) in enumerate(held):
            n = len(w)
            assert srv.wait(t, 60000.0)["state"] == 2
            anc = torch.zeros(n, dtype=torch.int32, device="cuda")
            out = torch.zeros((n, d), device="cuda")
            mgp.mgp_server_copy_outputs(srv.handle, t, anc.data_ptr(), out.data_ptr(), mgp.current_stream())
            torch.cuda.synchronize()
            B = oracle.B_from_weights(w, 0.01)[0] if f % 2 else 23
            ref = oracle.resample(w, "megopolis", B, 6, stream_id=f)
            np.testing.assert_array_equal(anc.cpu().numpy(), ref)
            np.testing.assert_array_equal(out.cpu().numpy(), st.reshape(n, d)[ref])
            srv.release(t)
    finally:
        srv.close()
