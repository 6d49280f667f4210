"""The stream that a call without one goes to: torch's current stream, through
torch's own functions for it where they are there and through its public
interface where they are not."""
from types import SimpleNamespace

import pytest

from paper_2203_04158_amd import binding


def _torch(raw, initialized=True):
    c = SimpleNamespace()
    if raw:
        c._cuda_getDevice = lambda: 3
        c._cuda_getCurrentRawStream = lambda device: 1000 + device
    cuda = SimpleNamespace(is_initialized=lambda: initialized, current_stream=lambda: SimpleNamespace(cuda_stream=77))
    return SimpleNamespace(_C=c, cuda=cuda)


@pytest.mark.parametrize("raw,initialized,want", [(True, True, 1003), (True, False, 77), (False, True, 77), (False, False, 77)])
def test_current_stream_with_and_without_private_functions(monkeypatch, raw, initialized, want):
    fake = _torch(raw, initialized)
    monkeypatch.setattr(binding, "_T", fake)
    monkeypatch.setattr(binding, "_raw_stream", binding._find_raw_stream(fake))
    assert binding._stream(None) == want
    assert binding._stream(5) == 5 and binding._stream(SimpleNamespace(cuda_stream=6)) == 6


def test_one_missing_function_is_enough():
    fake = _torch(True)
    del fake._C._cuda_getDevice
    assert binding._find_raw_stream(fake) is None


@pytest.mark.gpu
def test_raw_and_public_streams_agree(monkeypatch):
    torch = pytest.importorskip("torch")
    torch.cuda.init()
    binding.lib()
    side = torch.cuda.Stream()
    for s in (torch.cuda.default_stream(), side):
        with torch.cuda.stream(s):
            raw = binding._stream(None)
            with monkeypatch.context() as m:
                m.setattr(binding, "_raw_stream", None)
                assert binding._stream(None) == raw == s.cuda_stream
