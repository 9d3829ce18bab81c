"""The stream a call is enqueued on is torch's current one at the time of the call: default, side stream, per thread."""
import threading

import pytest
import torch

from paper_2311_14272_amd import crisp

pytestmark = pytest.mark.gpu


def test_current_stream_is_asked_for_on_every_call():
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    assert crisp._stream() == (torch.cuda.current_stream().cuda_stream or None)
    with torch.cuda.stream(side):
        assert crisp._stream() == side.cuda_stream
        with torch.cuda.stream(other):
            assert crisp._stream() == other.cuda_stream
        seen = []
        t = threading.Thread(target=lambda: seen.append(crisp._stream()))   # a thread has a current stream of its own
        t.start()
        t.join()
        assert seen == [None]
        assert crisp._stream() == side.cuda_stream
    assert crisp._stream() is None
