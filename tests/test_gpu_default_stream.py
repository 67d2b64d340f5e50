"""The stream that a call without a stream argument is enqueued on."""
import pytest


@pytest.mark.gpu
def test_default_stream_handle_is_that_of_the_current_stream():
    """What a call without a stream argument is enqueued on: the calling thread's current stream, inside a stream context and
    outside of it."""
    import threading

    import torch
    from paper_2508_06001_amd import binding as B
    other = torch.cuda.Stream()
    seen = []

    def look():
        seen.append((B._stream_handle(None), int(torch.cuda.current_stream().cuda_stream)))

    look()
    with torch.cuda.stream(other):
        look()
        t = threading.Thread(target=look)
        t.start()
        t.join()
    look()
    assert all(a == b for a, b in seen) and seen[1][0] == int(other.cuda_stream) != seen[0][0], seen
