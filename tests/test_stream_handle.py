"""The binding's default stream: torch's current stream on the current device,
by the raw-handle calls where this torch has them and by its public interface
where it has not."""
import pytest
import torch

from paper_1802_00930_amd import dfp


class _Stream:
    cuda_stream = 0x1234


def test_without_raw_handle_calls(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_stream", _Stream)
    for name in ("_raw_stream", "_device"):
        with monkeypatch.context() as m:
            m.setattr(dfp, name, None)
            assert dfp._stream(None) == 0x1234
    assert dfp._stream(_Stream()) == 0x1234


@pytest.mark.gpu
def test_raw_handle_is_the_current_stream(monkeypatch):
    side = torch.cuda.Stream()
    for ctx in (torch.cuda.stream(side), torch.cuda.stream(torch.cuda.default_stream())):
        with ctx:
            assert dfp._stream(None) == torch.cuda.current_stream().cuda_stream
            with monkeypatch.context() as m:
                m.setattr(dfp, "_raw_stream", None)
                assert dfp._stream(None) == torch.cuda.current_stream().cuda_stream
    assert dfp._stream(side) == side.cuda_stream
