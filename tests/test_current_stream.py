"""redsum.current_stream() without a GPU: torch's raw handle where torch has
the raw accessors, its public stream object where either is missing (they are
not public) and before torch's CUDA state exists."""
import types

import pytest

from paper_2004_05371_amd import redsum

torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def fake_streams(monkeypatch):
    monkeypatch.setattr(redsum, "_raw_stream", None)
    monkeypatch.setattr(redsum, "_raw_device", None)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=7))
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda dev: 100 + dev, raising=False)


def test_raw_handle_of_the_current_device():
    assert redsum.current_stream() == 103 and redsum.current_stream() == 103


@pytest.mark.parametrize("name", ["_cuda_getDevice", "_cuda_getCurrentRawStream"])
def test_public_stream_where_torch_has_no_raw_accessor(monkeypatch, name):
    monkeypatch.delattr(torch._C, name)
    assert redsum.current_stream() == 7 and redsum.current_stream() == 7


def test_public_stream_before_initialization(monkeypatch):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: False)
    assert redsum.current_stream() == 7
