"""A call without a stream argument goes to torch's current stream: the default one, one made current, and back again."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_current_stream_handle():
    from paper_2605_07330_amd import srs
    side = torch.cuda.Stream()
    assert srs._stream_ptr(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert srs._stream_ptr(None) == side.cuda_stream == srs._stream_ptr(side)
    assert srs._stream_ptr(None) == torch.cuda.current_stream().cuda_stream
