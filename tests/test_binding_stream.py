"""The stream that calls are enqueued on is torch's current one, with and without the functions of torch that give it without a Stream object."""
import types

import pytest
import torch

from paper_2509_25149_amd import binding as nv


def test_without_torchs_raw_functions(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=1234))
    for missing in (types.SimpleNamespace(), types.SimpleNamespace(_cuda_getDevice=lambda: 0), types.SimpleNamespace(_cuda_getCurrentRawStream=lambda d: 7)):
        assert nv._stream_getter(missing)() == 1234
    assert nv._stream_getter(types.SimpleNamespace(_cuda_getDevice=lambda: 3, _cuda_getCurrentRawStream=lambda d: 70 + d))() == 73


@pytest.mark.gpu
def test_current_stream():
    assert nv._stream() == torch.cuda.current_stream().cuda_stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert nv._stream() == s.cuda_stream == nv._stream_getter(types.SimpleNamespace())()
    assert nv._stream() == torch.cuda.current_stream().cuda_stream
