"""The gather on both sides of 2^31 elements, where its row numbers change from
32-bit multiplications to 64-bit divisions, and the multiplications near that end
for many row lengths: every output row against torch's own indexing (copies: no
tolerance)."""
import pytest

pytestmark = pytest.mark.gpu
CHUNK = 1 << 25  # rows compared at once


def _check(d, n_out, n_states, seed):
    import torch

    from paper_2109_13504_amd import mgp
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    states = torch.randn((n_states, d), generator=g, device="cuda")
    anc = torch.randint(0, n_states, (n_out,), generator=g, device="cuda", dtype=torch.int32)
    out = torch.empty((n_out, d), device="cuda")
    mgp.gather(states, anc, out=out)
    step = max(1, CHUNK // d)
    # every row where there are few, else the first and last ones and some between
    starts = range(0, n_out, step) if n_out <= 64 * step else [0, n_out // 3, n_out // 2, n_out - 2 * step, n_out - step]
    for a in starts:
        b = min(n_out, a + step)
        assert torch.equal(out[a:b], states[anc[a:b].long()]), f"rows {a} to {b} of {n_out}, d = {d}"
    del out, anc
    torch.cuda.empty_cache()


@pytest.mark.parametrize("d,n_out", [
    (1, (1 << 31) - 1),                # the most outputs there are: below 2^31 floats
    (3, 715827882), (3, 715827883),    # 2^31 - 2 and 2^31 + 1 floats
    (8, (1 << 30) - 1), (8, 1 << 30),  # 2^31 - 2 and 2^31 float4s
])
def test_around_2pow31_elements(d, n_out):
    _check(d, n_out, 1009, d)


@pytest.mark.parametrize("d", [2, 5, 7, 13, 33, 100, 127, 129, 641, 1000, 4097, 65535, 65537, (1 << 20) + 1,
                               (1 << 24) - 1, (1 << 24) + 4])
def test_row_lengths_near_the_end(d):
    """The last whole rows below 2^31 floats (float4s for the last length)."""
    _check(d, min(((1 << 31) - 1) // d, (1 << 28)), 5, d)


@pytest.mark.parametrize("d,n_out", [(4, (5 << 19) - 1), (4, 5 << 19), (12, 873813), (12, 873814), (4, 1 << 24),
                                     (4, (1 << 24) + 1), (20, 3355443), (20, 3355444), (16, 1 << 22)])
def test_float4s_per_thread(d, n_out):
    """On both sides of the numbers of float4s where a thread takes one, not two."""
    _check(d, n_out, 100003, d)
