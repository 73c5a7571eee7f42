"""mgp_gather with element numbers divided by multiplication: every copied word
against torch indexing (exact) for row lengths of one to many floats, whole and
ragged last blocks, both numbers of elements per thread, bases with and without
16-byte alignment, and NaN rows for ancestors out of range."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 7, 8, 12, 31, 33, 64, 127, 129])
@pytest.mark.parametrize("n_out", [1, 255, 512, 1025, 70001])
def test_rows(d, n_out):
    import torch

    from paper_2109_13504_amd import mgp
    n_states = 3001
    g = torch.Generator().manual_seed(d * 1000 + n_out)
    base = torch.randn(n_states * d + 1, generator=g).cuda()
    anc = torch.randint(0, n_states, (n_out,), generator=g, dtype=torch.int32).cuda()
    for shift in (0, 1):
        st = base[shift:shift + n_states * d].view(n_states, d)
        np.testing.assert_array_equal(mgp.gather(st, anc).cpu().numpy(), st[anc.long()].cpu().numpy())
    bad = anc.clone()
    bad[0], bad[-1] = -1, n_states
    got = mgp.gather(st, bad).cpu().numpy()
    ref = st[bad.long().clamp(0, n_states - 1)].cpu().numpy()
    ref[0], ref[-1] = np.nan, np.nan
    np.testing.assert_array_equal(got, ref)


@pytest.mark.parametrize("d", [3, 8, 1023])
def test_large(d):
    """Element numbers up to 2^30 and more."""
    import torch

    from paper_2109_13504_amd import mgp
    n_out, n_states = ((1 << 30) + 12345) // d, 257
    st = torch.randn(n_states, d, device="cuda")
    anc = torch.randint(0, n_states, (n_out,), dtype=torch.int32, device="cuda")
    got = mgp.gather(st, anc)
    for a in range(0, n_out, max(1, n_out // 7)):
        e = min(n_out, a + 5000)
        assert torch.equal(got[a:e], st[anc[a:e].long()])
    assert torch.equal(got[-1000:], st[anc[-1000:].long()])
