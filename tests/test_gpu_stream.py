"""Calls without a stream go to the current stream of the calling thread's current device."""
import threading

import pytest
import torch

from paper_2506_01380_amd import binding as nb

pytestmark = pytest.mark.gpu


def test_default_stream_is_the_threads_current_one():
    assert nb._stream(None) == torch.cuda.current_stream().cuda_stream
    s, seen = torch.cuda.Stream(), {}
    with torch.cuda.stream(s):
        assert nb._stream(None) == s.cuda_stream != 0
        t = threading.Thread(target=lambda: seen.setdefault("other", nb._stream(None)))
        t.start()
        t.join()
    assert nb._stream(None) == torch.cuda.current_stream().cuda_stream != s.cuda_stream
    assert seen["other"] == torch.cuda.default_stream().cuda_stream
    assert nb._stream(s) == s.cuda_stream and nb._stream(7) == 7
