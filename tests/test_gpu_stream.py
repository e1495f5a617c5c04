"""Calls without a stream argument run on torch's current stream: the handle the binding takes is the current one's."""
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu


def test_current_stream_handle():
    if not gpu_available():
        pytest.skip("no GPU")
    import threading

    import torch
    from paper_2608_15602_amd import fluxbin as fb
    assert fb._stream(None) == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert fb._stream(None) == side.cuda_stream
        other = []
        t = threading.Thread(target=lambda: other.append((fb._stream(None), torch.cuda.current_stream().cuda_stream)))
        t.start()
        t.join()
        assert other[0][0] == other[0][1]   # the current stream is a thread's own
    assert fb._stream(None) == torch.cuda.current_stream().cuda_stream
    assert fb._stream(side) == side.cuda_stream and fb._stream(side.cuda_stream) == side.cuda_stream
