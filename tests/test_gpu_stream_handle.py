"""The stream a call without one is launched on: torch's current stream of the calling thread, inside and outside a stream
context, in another thread, and an explicit one."""
import threading

import pytest

pytestmark = pytest.mark.gpu


def test_current_stream_of_the_thread():
    import torch
    import paper_2512_03383_amd as uq
    side, seen = torch.cuda.Stream(), []
    torch.zeros(1, device="cuda")

    def handle(stream=None):
        return uq._stream_ptr(stream)

    assert handle() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert handle() == side.cuda_stream == torch.cuda.current_stream().cuda_stream
        t = threading.Thread(target=lambda: seen.append((handle(), torch.cuda.current_stream().cuda_stream)))
        t.start()
        t.join()
        assert seen[0][0] == seen[0][1]
    assert handle(side) == side.cuda_stream and handle() != side.cuda_stream
