"""Calls without a stream run on the caller's current stream, asked for at each
call: the default one, one set by a context, and each thread's own."""
import threading

import pytest

pytestmark = pytest.mark.gpu


def test_current_stream_is_asked_for():
    import torch
    from paper_2411_10143_amd import _binding as B
    torch.cuda.init()

    def agrees():
        return B._stream(None) == torch.cuda.current_stream().cuda_stream

    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    assert agrees()
    with torch.cuda.stream(a):
        assert agrees() and B._stream(None) == a.cuda_stream
        with torch.cuda.stream(b):
            assert B._stream(None) == b.cuda_stream
            seen = []
            t = threading.Thread(target=lambda: seen.append((agrees(), B._stream(None))))
            t.start()
            t.join()
            assert seen == [(True, torch.cuda.default_stream().cuda_stream)]
        assert B._stream(None) == a.cuda_stream
    assert agrees()
    assert B._stream(a) == a.cuda_stream and B._stream(7) == 7
