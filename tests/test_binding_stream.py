"""Which of torch's calls give the current stream's handle: its private ones where they are there, else the
public one.  Host code; torch is replaced by stand-ins."""
import types

import pytest
import torch

from paper_2511_12653_amd import binding


@pytest.mark.parametrize("missing", [(), ("_cuda_getCurrentRawStream",), ("_cuda_getDevice",)])
def test_stream_lookup(monkeypatch, missing):
    private = {"_cuda_getCurrentRawStream": lambda device: 0x100 + device, "_cuda_getDevice": lambda: 3}
    monkeypatch.setattr(torch, "_C", types.SimpleNamespace(**{k: v for k, v in private.items() if k not in missing}))
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x777))
    assert binding._stream_lookup()() == (0x777 if missing else 0x103)
