"""The stream handle comes from torch's public interface where the quicker private one is absent."""
from types import SimpleNamespace

import pytest
import torch

from paper_2601_05732_amd import binding


@pytest.mark.parametrize("absent", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_without_the_private_functions(monkeypatch, absent):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=4711))
    monkeypatch.delattr(torch._C, absent, raising=False)
    assert binding._stream() == 4711
