"""Where the binding takes the current device and stream from."""
import types

import pytest
import torch

from paper_2604_19906_amd import tpo


@pytest.fixture
def fresh(monkeypatch):
    monkeypatch.setattr(tpo, "_rt", None)


@pytest.mark.parametrize("missing", ["_cuda_getDevice", "_cuda_getCurrentRawStream"])
def test_public_calls_stand_in_for_private_ones(fresh, monkeypatch, missing):
    """A torch without the private functions must not stop a call."""
    monkeypatch.delattr(torch._C, missing)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda dev: types.SimpleNamespace(cuda_stream=100 + dev))
    codes, device, stream = tpo._runtime()
    assert codes == {torch.float64: tpo.TPO_F64, torch.float32: tpo.TPO_F32}
    assert stream(device()) == 103


@pytest.mark.gpu
def test_both_name_the_same_stream(fresh):
    other = torch.cuda.Stream()
    _, device, stream = tpo._runtime()
    for s in (torch.cuda.current_stream(), other):
        with torch.cuda.stream(s):
            assert device() == torch.cuda.current_device()
            assert stream(device()) == torch.cuda.current_stream().cuda_stream == s.cuda_stream
