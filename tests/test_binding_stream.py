"""CPU: which stream the binding launches on when the caller names none, with stand-ins for torch."""
from types import SimpleNamespace

import pytest

from paper_2412_01523_amd import binding as fx


def torch_with(private, initialized):
    cuda = SimpleNamespace(is_initialized=lambda: initialized, current_stream=lambda: SimpleNamespace(cuda_stream=77))
    table = {"_cuda_getCurrentRawStream": lambda device: 100 + device, "_cuda_getDevice": lambda: 3}
    return SimpleNamespace(cuda=cuda, _C=SimpleNamespace(**{n: table[n] for n in private}))


@pytest.mark.parametrize("private,initialized,want", [
    (("_cuda_getCurrentRawStream", "_cuda_getDevice"), True, 103),
    (("_cuda_getCurrentRawStream", "_cuda_getDevice"), False, 77),   # nothing to ask before torch has started the GPU
    (("_cuda_getCurrentRawStream",), True, 77), (("_cuda_getDevice",), True, 77), ((), True, 77),
])
def test_current_stream(private, initialized, want, monkeypatch):
    monkeypatch.setattr(fx, "_current_stream", fx._current_stream_of(torch_with(private, initialized)))
    assert fx._stream(None) == want
    assert fx._stream(5) == 5 and fx._stream(SimpleNamespace(cuda_stream=9)) == 9
