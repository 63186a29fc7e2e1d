"""Where the handle of the current stream comes from."""
import types

from paper_2104_10231_amd import relres


def test_private_entries_are_optional(monkeypatch):
    """Without the entries of torch._C (or with one of them) the public call
    serves, and a given stream's own handle always does."""
    stream = types.SimpleNamespace(cuda_stream=4711)
    monkeypatch.setattr(relres.torch.cuda, "current_stream", lambda: stream)
    for core in (types.SimpleNamespace(), types.SimpleNamespace(_cuda_getDevice=lambda: 3)):
        monkeypatch.setattr(relres, "_current_stream", relres._current_stream_reader(core))
        assert relres._stream(None) == 4711
    core = types.SimpleNamespace(_cuda_getDevice=lambda: 3, _cuda_getCurrentRawStream=lambda d: 100 + d)
    monkeypatch.setattr(relres, "_current_stream", relres._current_stream_reader(core))
    assert relres._stream(None) == 103
    assert relres._stream(types.SimpleNamespace(cuda_stream=9)) == 9
