"""The stream handle of a call where torch lacks its private shortcut: the
public API's.  No GPU is used."""
import importlib.util
import types

import pytest

torch = pytest.importorskip("torch")
soax = pytest.importorskip("paper_1710_03462_amd")


def test_public_handle_without_the_private_name(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda: types.SimpleNamespace(cuda_stream=0x1234))
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    # a copy of the module of its own, imported without the name
    spec = importlib.util.spec_from_file_location("paper_1710_03462_amd._particles_copy",
                                                  soax.particles.__file__)
    copy = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(copy)
    assert copy.stream_handle() == 0x1234
    assert copy.current_stream().value == 0x1234
