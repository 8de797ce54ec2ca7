"""Calls go to torch's current stream, whichever it is."""
import threading

import pytest
import torch

from paper_2508_17588_amd import binding

pytestmark = pytest.mark.gpu


def test_the_stream_handed_over_is_the_current_one():
    side = torch.cuda.Stream()
    assert (binding._stream().value or 0) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert binding._stream().value == side.cuda_stream != 0
        seen = []                       # another thread has a current stream of its own
        t = threading.Thread(target=lambda: seen.append(binding._stream().value or 0))
        t.start()
        t.join()
        assert seen == [torch.cuda.default_stream().cuda_stream]
    assert (binding._stream().value or 0) == torch.cuda.default_stream().cuda_stream
