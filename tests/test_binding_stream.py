"""The binding's stream query: the raw handle where torch hands it out, the public call where it does not."""
import types

import pytest
import torch

from paper_2508_07101_amd import binding as cb


class _Cuda:
    def __init__(self, initialized=True):
        self._initialized = initialized

    def is_initialized(self):
        return self._initialized

    def current_stream(self):
        return types.SimpleNamespace(cuda_stream=77)


@pytest.mark.parametrize("names", [(), ("_cuda_getCurrentRawStream",), ("_cuda_getDevice",)])
def test_a_torch_without_the_raw_stream_query_is_served_by_the_public_call(names):
    c = types.SimpleNamespace(**{n: (lambda *a: 5) for n in names})
    assert cb.stream_query(types.SimpleNamespace(_C=c, cuda=_Cuda()))() == 77


def test_the_raw_handle_of_the_current_device_is_used_once_a_device_is_up():
    asked = []
    c = types.SimpleNamespace(_cuda_getDevice=lambda: 3, _cuda_getCurrentRawStream=lambda dev: asked.append(dev) or 9)
    assert cb.stream_query(types.SimpleNamespace(_C=c, cuda=_Cuda()))() == 9 and asked == [3]
    assert cb.stream_query(types.SimpleNamespace(_C=c, cuda=_Cuda(initialized=False)))() == 77


@pytest.mark.gpu
def test_the_query_names_the_current_stream():
    torch.cuda.init()
    assert cb._stream() == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert cb._stream() == side.cuda_stream
    assert cb._stream() == torch.cuda.current_stream().cuda_stream
