"""Calls are enqueued on torch's current stream, whichever that is."""
import pytest

pytestmark = pytest.mark.gpu


def test_current_stream_is_used():
    import torch
    from paper_2311_12023_amd import lq
    assert lq._stream() == torch.cuda.current_stream().cuda_stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert lq._stream() == s.cuda_stream == torch.cuda.current_stream().cuda_stream
    assert lq._stream() == torch.cuda.current_stream().cuda_stream
