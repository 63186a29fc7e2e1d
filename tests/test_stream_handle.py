"""Where the handle of the current stream comes from."""
import types

from paper_2104_10231_amd import relres


def test_private_entries_are_optional(monkeypatch):
    """Without the entries of torch._C (or with one of them) the public call
    serves, and a given stream's own handle always does."""
    stream = types.SimpleNamespace(cuda_stream=4711)
    monkeypatch.setattr(relres.torch.cuda, "current_stream", lambda: stream)
    for core, want in ((types.SimpleNamespace(), 4711),
                       (types.SimpleNamespace(_cuda_getDevice=lambda: 3), 4711),
                       (types.SimpleNamespace(_cuda_getDevice=lambda: 3,
                                              _cuda_getCurrentRawStream=lambda d: 100 + d), 103)):
        for name, value in zip(("_raw_stream", "_device"), relres._stream_readers(core)):
            monkeypatch.setattr(relres, name, value)
        assert relres._stream(None) == want
        assert relres._stream(types.SimpleNamespace(cuda_stream=9)) == 9
