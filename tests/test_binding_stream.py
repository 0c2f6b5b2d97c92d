"""Host-only: the stream handle that the binding passes on, with and without torch's own short way to it."""
import types

import pytest
import torch

from paper_2603_09983_amd import binding as B


@pytest.mark.parametrize("missing", ["_raw_stream", "_current_device", None])
def test_current_stream(monkeypatch, missing):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    monkeypatch.setattr(B, "_raw_stream", lambda dev: 70 + dev)
    monkeypatch.setattr(B, "_current_device", lambda: 7)
    if missing:
        monkeypatch.setattr(B, missing, None)
    assert B._stream(None) == 77
    assert B._stream(types.SimpleNamespace(cuda_stream=5)) == 5 and B._stream(9) == 9
