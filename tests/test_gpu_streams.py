"""The stream handle that a call passes to the library is torch's current one:
on the default stream, under a stream context, in another thread, and while a
graph is captured; and the workspaces follow it."""
import threading

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_current_stream_handle():
    from paper_2202_10297_amd import ops

    dev = torch.zeros(1, device="cuda").device
    seen = []

    def look():
        want = torch.cuda.current_stream(dev).cuda_stream
        seen.append(want)
        assert ops._stream(dev) == want == ops._stream("cuda") == ops._stream()
        ws = ops.WS.get("stream test", 256, dev)
        assert ops.WS.get("stream test", 256, dev) is ws
        return ws

    s = torch.cuda.Stream()
    w0 = look()
    with torch.cuda.stream(s):
        assert look() is not w0
        t = threading.Thread(target=look)  # a thread starts on the default stream
        t.start()
        t.join()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        look()
    assert len(seen) == 4 and seen[0] == seen[2] != seen[1] and seen[3] != seen[0]
    assert look() is w0


def test_cpu_tensors_stay_refused():
    from paper_2202_10297_amd import ops

    with pytest.raises(ValueError):
        ops.linrec_scan(torch.ones(8), torch.ones(8))
