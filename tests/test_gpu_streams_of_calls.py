"""A call without a stream goes to the current stream, whichever that is from call to call."""
import pytest

from paper_2502_02789_amd import binding as sp

pytestmark = pytest.mark.gpu


def test_the_current_stream_is_looked_up_at_every_call():
    import torch
    for _ in range(2):
        assert sp._stream_handle(None) == (int(torch.cuda.current_stream().cuda_stream) or None)
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            assert sp._stream_handle(None) == int(side.cuda_stream)
        assert sp._stream_handle(None) == (int(torch.cuda.current_stream().cuda_stream) or None)
        assert sp._stream_handle(side) == int(side.cuda_stream)
