"""The binding enqueues on the caller's current stream, whichever that is."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_binding_uses_the_current_stream():
    from paper_2501_13986_amd import binding as b
    side = torch.cuda.Stream()
    external = torch.cuda.ExternalStream(torch.cuda.Stream().cuda_stream)
    for s in (torch.cuda.default_stream(), side, external, side):
        with torch.cuda.stream(s):
            assert b._stream() == torch.cuda.current_stream().cuda_stream == s.cuda_stream
            with torch.cuda.device(0):
                assert b._stream() == s.cuda_stream
    assert b._stream() == torch.cuda.default_stream().cuda_stream
    seen = []
    import threading
    def other():   # the current stream is a thread's own
        seen.append(b._stream())
        with torch.cuda.stream(side):
            seen.append(b._stream())
    t = threading.Thread(target=other)
    with torch.cuda.stream(external):
        t.start()
        t.join()
    assert seen == [torch.cuda.default_stream().cuda_stream, side.cuda_stream]
