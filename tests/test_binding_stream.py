"""The binding asks torch for the current stream's handle without a Stream object where this torch has the names for that, and through
the public one where it has not."""
import types

import pytest

torch = pytest.importorskip("torch")

from paper_2605_21226_amd import binding  # noqa: E402


@pytest.mark.parametrize("missing", [("_cuda_getCurrentRawStream",), ("_cuda_getDevice",), ("_cuda_getCurrentRawStream", "_cuda_getDevice")])
def test_current_stream_without_the_private_names(monkeypatch, missing):
    handles = iter([11, 12, 13])
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=next(handles)))
    monkeypatch.setattr(binding, "_raw_stream", None)
    monkeypatch.setattr(binding, "_device", None)
    for name in missing:
        monkeypatch.delattr(torch._C, name, raising=False)
    assert [binding._stream_ptr(None), binding._stream_ptr(None)] == [12, 13]      # (the first one asks whether there is a device)
    assert binding._stream_ptr(types.SimpleNamespace(cuda_stream=5)) == 5
