"""The stream that a call of the binding takes where none is given: the calling thread's current one."""
import threading

import pytest
import torch

from paper_2404_19124_amd import binding as B

pytestmark = pytest.mark.gpu


def test_current_stream_of_the_calling_thread():
    torch.cuda.init()
    side = torch.cuda.Stream()
    default = torch.cuda.current_stream().cuda_stream
    assert B._stream_ptr(None) == default
    seen = []
    with torch.cuda.stream(side):
        assert B._stream_ptr(None) == side.cuda_stream != default
        other = threading.Thread(target=lambda: seen.append(B._stream_ptr(None)))
        other.start()
        other.join()
    assert seen == [default]
    assert B._stream_ptr(None) == default and B._stream_ptr(side) == side.cuda_stream
