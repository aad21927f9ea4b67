"""The handle of the current stream: through torch's own functions where it has them, through a Stream object where not."""
import types

from paper_2512_19206_amd import binding


def test_current_stream(monkeypatch):
    import torch
    stream = types.SimpleNamespace(cuda_stream=77)
    assert binding._stream_ptr(stream) == 77
    monkeypatch.setattr(binding, "_device", lambda: 3)
    monkeypatch.setattr(binding, "_raw_stream", lambda device: 100 + device)
    assert binding._stream_ptr(None) == 103
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: stream)
    for name in ("_device", "_raw_stream"):
        with monkeypatch.context() as m:
            m.setattr(binding, name, None)
            assert binding._stream_ptr(None) == 77
