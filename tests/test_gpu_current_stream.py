"""Calls without a stream go to the current one, whichever that is."""
import threading

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1705_09776_amd as cd  # noqa: E402


def test_the_handle_is_the_current_streams():
    assert cd._stream(None) == torch.cuda.default_stream().cuda_stream
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    assert cd._stream(a) == a.cuda_stream and cd._stream(a.cuda_stream) == a.cuda_stream
    with torch.cuda.stream(a):
        assert cd._stream(None) == a.cuda_stream
        with torch.cuda.stream(b):
            assert cd._stream(None) == b.cuda_stream
        got = []
        t = threading.Thread(target=lambda: got.append(cd._stream(None)))   # a thread has its own current stream
        t.start()
        t.join()
        assert got == [torch.cuda.default_stream().cuda_stream]
        assert cd._stream(None) == a.cuda_stream
    ext = torch.cuda.ExternalStream(b.cuda_stream)
    with torch.cuda.stream(ext):
        assert cd._stream(None) == b.cuda_stream
    g = torch.cuda.CUDAGraph()
    x = torch.zeros(4, device="cuda")
    with torch.cuda.graph(g):
        x.add_(1)
        inside, want = cd._stream(None), torch.cuda.current_stream().cuda_stream
    assert inside == want != torch.cuda.default_stream().cuda_stream
