"""The stream a call without one goes to: torch's current stream, whichever is current where the call is made."""

import pytest

from paper_2001_00138_amd import binding as B

pytestmark = pytest.mark.gpu


def test_calls_go_to_the_current_stream():
    import threading

    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    side = torch.cuda.Stream()
    seen = {}

    def look(name):
        seen[name] = (B._stream_ptr(None), torch.cuda.current_stream().cuda_stream or None)

    look("default")
    with torch.cuda.stream(side):
        look("side")
        other = threading.Thread(target=look, args=("thread",))       # a thread has a current stream of its own
        other.start()
        other.join()
        with torch.cuda.stream(torch.cuda.default_stream()):
            look("nested")
    look("after")
    assert all(a == b for a, b in seen.values())
    assert seen["side"][0] == side.cuda_stream != seen["default"][0]
    assert B._stream_ptr(side) == B._stream_ptr(side.cuda_stream) == side.cuda_stream and B._stream_ptr(0) is None
