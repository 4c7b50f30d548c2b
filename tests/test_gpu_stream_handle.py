"""The stream that a call without one is enqueued on is torch's current stream, whatever that is."""
import pytest
import torch

from paper_2604_20470_amd import binding

pytestmark = pytest.mark.gpu


def test_default_is_the_current_stream():
    handle = lambda: binding._stream(None).value or 0
    side = torch.cuda.Stream()
    assert handle() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert handle() == side.cuda_stream == torch.cuda.current_stream().cuda_stream
    assert handle() == torch.cuda.current_stream().cuda_stream
    assert binding._stream(side).value == side.cuda_stream and binding._stream(side.cuda_stream).value == side.cuda_stream
