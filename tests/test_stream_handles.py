"""Which stream a call's handle is of (on the CPU, with torch's stream functions replaced)."""

import types

import pytest
import torch

from paper_2604_06257_amd import das


@pytest.mark.parametrize("raw", [True, False])
def test_current_stream_with_and_without_torchs_raw_handle(raw, monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=1003))
    monkeypatch.setattr(das, "_raw_stream", (lambda device: 1000 + device) if raw else None)
    for none in (None, 0):
        assert das._stream_ptr(none) == 1003
    assert das._stream_ptr(types.SimpleNamespace(cuda_stream=77)) == 77
