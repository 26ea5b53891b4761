"""Calls without a stream argument go to the current stream of the current device: the handle is torch's own."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_default_stream_argument_follows_the_current_stream():
    from paper_2605_15250_amd import binding as B
    side = torch.cuda.Stream()
    for _ in range(2):   # the first call resolves the entry, the second uses it
        assert B._stream(None) == torch.cuda.current_stream().cuda_stream
        with torch.cuda.stream(side):
            assert B._stream(None) == side.cuda_stream == torch.cuda.current_stream().cuda_stream
        assert B._stream(side) == side.cuda_stream and B._stream(17) == 17
    B._forget_raw_stream()   # what a forked child starts from
    assert B._stream(None) == torch.cuda.current_stream().cuda_stream
