"""The stream that a call without one goes to is torch's current stream, as
torch.cuda.current_stream() names it: the default one, a side stream, another
thread's, and a capturing one."""
import threading

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _same():
    import paper_2601_07892_amd as sh
    return (sh._stream(None) or 0) == torch.cuda.current_stream().cuda_stream


def test_current_stream():
    import paper_2601_07892_amd as sh
    torch.zeros(1, device="cuda")
    assert _same() and sh._stream(1234) == 1234
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert _same() and sh._stream(None) == side.cuda_stream
        got = []
        th = threading.Thread(target=lambda: got.append((_same(), sh._stream(None) or 0)))
        th.start()
        th.join()
        assert got[0][0] and got[0][1] != side.cuda_stream  # another thread: its own
    assert _same()


def test_without_the_raw_handle(monkeypatch):
    import paper_2601_07892_amd as sh
    torch.zeros(1, device="cuda")
    monkeypatch.setattr(sh, "_raw_stream", None)
    with torch.cuda.stream(torch.cuda.Stream()):
        assert _same()


def test_capture():
    import paper_2601_07892_amd as sh
    x = torch.randn(3, 256, device="cuda")
    q = torch.empty(3, 256, dtype=torch.int8, device="cuda")
    sx = torch.empty(3, device="cuda")
    sh.sherry_quantize_act(x, q, sx)
    torch.cuda.synchronize()
    want = q.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        assert _same()
        sh.sherry_quantize_act(x, q, sx)
    for _ in range(3):
        q.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(q, want)
