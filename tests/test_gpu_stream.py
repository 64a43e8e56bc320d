"""Calls without a stream go to the calling thread's current one, on the default stream, inside a stream block and in another
thread (whose current stream is the default one whatever this thread has set)."""
import threading

import pytest
import torch

from paper_2510_06710_amd import binding as vb

pytestmark = pytest.mark.gpu


def test_current_stream():
    torch.zeros(1, device="cuda:0")
    assert vb._stream(None) == (torch.cuda.current_stream().cuda_stream or None)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert vb._stream(None) == side.cuda_stream
        seen = []
        t = threading.Thread(target=lambda: seen.append((vb._stream(None), torch.cuda.current_stream().cuda_stream or None)))
        t.start()
        t.join()
        assert seen[0][0] == seen[0][1]
    assert vb._stream(side) == side.cuda_stream
