"""The stream handle that the binding passes, without a device: torch's raw
handle where this torch has the call, its Stream object otherwise."""
import types

import pytest

from paper_1011_3318_amd import wcl as W


class FakeStream:
    cuda_stream = 77


@pytest.mark.parametrize("missing", [(), ("_cuda_getCurrentRawStream",), ("_cuda_getDevice",),
                                     ("_cuda_getCurrentRawStream", "_cuda_getDevice")])
def test_current_stream_with_and_without_the_raw_call(monkeypatch, missing):
    raw = {"_cuda_getCurrentRawStream": lambda dev: 77, "_cuda_getDevice": lambda: 0}
    cuda = types.SimpleNamespace(is_initialized=lambda: True, current_stream=lambda: FakeStream,
                                 Stream=W.torch.cuda.Stream)
    c = types.SimpleNamespace(**{k: f for k, f in raw.items() if k not in missing})
    monkeypatch.setattr(W, "torch", types.SimpleNamespace(_C=c, cuda=cuda))
    assert W._stream(None) == 77
    assert W._stream(5) == 5
