"""The stream that a call runs on: the raw handle where torch has both functions that it takes, else the public way.  CPU only."""
from types import SimpleNamespace as NS

import pytest

from paper_2503_05840_amd import binding


def _torch(initialized=True, **private):
    return NS(_C=type("C", (), {k: staticmethod(v) for k, v in private.items()}),
              cuda=type("cuda", (), {"is_initialized": staticmethod(lambda: initialized), "current_stream": staticmethod(lambda: NS(cuda_stream=7))}))


RAW = {"_cuda_getCurrentRawStream": lambda device: 100 + device, "_cuda_getDevice": lambda: 3}


@pytest.mark.parametrize("names,initialized,handle", [
    (("_cuda_getCurrentRawStream", "_cuda_getDevice"), True, 103), (("_cuda_getCurrentRawStream", "_cuda_getDevice"), False, 7),
    (("_cuda_getCurrentRawStream",), True, 7), (("_cuda_getDevice",), True, 7), ((), True, 7),
])
def test_handle_of_the_current_stream(names, initialized, handle):
    class Hashable(NS):
        __hash__ = object.__hash__
    t = _torch(initialized, **{n: RAW[n] for n in names})
    assert binding._current_stream(Hashable(**vars(t)))() == handle
