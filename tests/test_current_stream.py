"""The current stream's handle: by torch's raw call where it has one, else from
its Stream object. (A stand-in for torch: no GPU needed.)"""
import types

import pytest

from paper_2109_13504_amd import mgp


@pytest.mark.parametrize("has_raw", [True, False])
def test_current_stream(monkeypatch, has_raw):
    c = types.SimpleNamespace()
    if has_raw:
        c._cuda_getCurrentRawStream = lambda device: 1000 + device
    cuda = types.SimpleNamespace(current_device=lambda: 3,
                                 current_stream=lambda: types.SimpleNamespace(cuda_stream=1003))
    monkeypatch.setattr(mgp, "_torch_module", types.SimpleNamespace(_C=c, cuda=cuda))
    assert mgp.current_stream() == 1003
