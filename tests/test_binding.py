"""Host side of the binding that needs no GPU."""
import types

import torch

import paper_2511_11430_amd as vpm


def test_current_stream_without_the_raw_handle(monkeypatch):
    """Without torch's handle getter, which is not a public name, the current Stream object's handle is used."""
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    assert vpm._stream(None) == 77
    assert vpm._stream(types.SimpleNamespace(cuda_stream=5)) == 5
