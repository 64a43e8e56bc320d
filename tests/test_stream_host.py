"""The binding's default stream without PyTorch's raw-stream functions, which are no public interface: the public call then gives it."""
from types import SimpleNamespace

import pytest
import torch

from paper_2510_06710_amd import binding as vb


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
@pytest.mark.parametrize("address", [0, 0x1230])
def test_a_pytorch_without_the_raw_functions(monkeypatch, missing, address):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=address))
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0x9990, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
    assert vb._stream(None) == 0x9990
    monkeypatch.delattr(torch._C, missing)
    assert vb._stream(None) == (address or None)
