"""A call without a stream goes to torch's current stream of the current device:
the handle looked up per call equals the Stream object's, on the default
stream, inside a stream context, nested, under capture and in another thread
(whose current stream is its own)."""
import threading

import pytest
import torch

from paper_2606_20537_amd import _native as N

pytestmark = pytest.mark.gpu


def test_current_stream_handle():
    torch.zeros(1, device="cuda")

    def same():
        assert N._stream(None) == torch.cuda.current_stream().cuda_stream
        return N._stream(None)

    default = same()
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    seen = []
    with torch.cuda.stream(a):
        assert same() == a.cuda_stream != default
        with torch.cuda.stream(b):
            assert same() == b.cuda_stream
        t = threading.Thread(target=lambda: seen.append(same()))
        t.start()
        t.join()
        assert same() == a.cuda_stream
    assert seen == [default] and same() == default
    x = torch.zeros(4, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=b):
        x.zero_()
        assert same() == b.cuda_stream
    torch.cuda.synchronize()
    assert N._stream(7) == 7 and N._stream(a) == a.cuda_stream
