"""The stream a call without one goes to: the calling thread's current stream
on the current device, the handle that torch.cuda.current_stream() holds."""
import threading

import pytest

pytestmark = pytest.mark.gpu


def test_default_stream_is_the_threads_current_one():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2404_00456_amd as q
    s, t = torch.cuda.Stream(), torch.cuda.Stream()
    assert q._stream(None) == torch.cuda.current_stream().cuda_stream
    assert q._stream(t) == t.cuda_stream
    seen = []
    with torch.cuda.stream(s):
        assert q._stream(None) == s.cuda_stream == torch.cuda.current_stream().cuda_stream
        th = threading.Thread(target=lambda: seen.append(
            (q._stream(None), torch.cuda.current_stream().cuda_stream)))
        th.start()
        th.join()
        with torch.cuda.stream(t):
            assert q._stream(None) == t.cuda_stream
        assert q._stream(None) == s.cuda_stream
    assert len(seen) == 1 and seen[0][0] == seen[0][1] != s.cuda_stream
