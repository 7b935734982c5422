"""The stream a call goes to: the one it is given, else the current device's
current one, in the default stream, inside a stream context, and in a thread
of its own (whose current stream is the default one)."""
import threading

import pytest

import paper_1012_2270_amd as rg

pytestmark = pytest.mark.gpu


def test_stream_of_a_call():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    assert side.cuda_stream != other.cuda_stream
    current = torch.cuda.current_stream().cuda_stream
    assert rg._stream() == rg._astream(None) == current
    seen = []
    with torch.cuda.stream(side):
        assert rg._stream() == rg._astream(None) == side.cuda_stream
        assert rg._stream(other) == rg._astream(None, other) == other.cuda_stream
        t = threading.Thread(target=lambda: seen.append((rg._stream(), torch.cuda.current_stream().cuda_stream)))
        t.start()
        t.join()
    assert seen[0][0] == seen[0][1]
    assert rg._stream() == current
