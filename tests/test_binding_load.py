"""What the loader does where the native binding cannot be used: it says so, and the Python form of the tensor functions stands
without it."""
import os

import pytest
import torch

from paper_2604_19906_amd import tpo


@pytest.fixture
def unloaded(monkeypatch):
    monkeypatch.setattr(tpo, "_native", None)


def refused():
    """The loader warns, and the functions run in their Python form."""
    with pytest.warns(UserWarning, match="Python form"):
        assert tpo._load_native() is False
    with pytest.raises(ValueError):
        tpo.apply_tensors(*[torch.zeros(1, 2, 2, 2)] * 5)


def test_binding_in_use_is_for_this_torch(unloaded):
    assert tpo._load_native().built_for == tpo.binding_versions()
    assert torch.__version__ in tpo.binding_versions()


@pytest.mark.parametrize("other", [("torch ", "torch 1."), ("cpython-", "cpython-9"), ("tpo.h ", "tpo.h 0")])
def test_binding_for_something_else_is_not_used(unloaded, monkeypatch, other):
    here = tpo.binding_versions()
    assert here.replace(*other) != here
    monkeypatch.setattr(tpo, "binding_versions", lambda: here.replace(*other))
    refused()


@pytest.mark.parametrize("content", [None, b"not a library"])
def test_missing_or_broken_binding(unloaded, monkeypatch, tmp_path, content):
    path = tmp_path / "_tpo_torch.so"
    if content is not None:
        path.write_bytes(content)
    monkeypatch.setattr(tpo, "TORCH_BINDING_PATH", os.fspath(path))
    refused()
