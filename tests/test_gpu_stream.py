"""The binding launches on torch's current stream of the calling thread, also after its first call."""
import threading

import pytest

pytestmark = pytest.mark.gpu


def test_current_stream_is_followed():
    import torch
    from paper_2605_26092_amd import binding
    current = lambda: torch.cuda.current_stream().cuda_stream
    assert binding._stream(None) == current()
    other, third = torch.cuda.Stream(), torch.cuda.Stream()
    for s in (other, third, other):
        with torch.cuda.stream(s):
            assert binding._stream(None) == s.cuda_stream
        assert binding._stream(None) == current()
    assert binding._stream(other) == other.cuda_stream and binding._stream(17) == 17
    with torch.cuda.stream(third):
        seen = []
        t = threading.Thread(target=lambda: seen.append((binding._stream(None), current())))     # (a thread has a current stream of its own)
        t.start()
        t.join()
        assert seen[0][0] == seen[0][1] and binding._stream(None) == third.cuda_stream
