"""The stream a call without one goes to, with and without torch's private shortcuts to its handle."""
import types

import pytest


@pytest.mark.parametrize("missing", [(), ("_cuda_getCurrentRawStream",), ("_cuda_getDevice",)])
def test_handle_of_the_current_stream(monkeypatch, missing):
    torch = pytest.importorskip("torch")
    from paper_2511_12056_amd import binding
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=4096 + 3))
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 4096 + device, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    for name in missing:
        monkeypatch.delattr(torch._C, name)
    assert binding._stream_handle(None) == 4096 + 3
    assert binding._stream_handle(types.SimpleNamespace(cuda_stream=0)) is None
