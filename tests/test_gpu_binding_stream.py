"""The binding launches on torch's current stream of the calling thread."""
import threading

import pytest

pytestmark = pytest.mark.gpu


def test_stream_is_torchs_current_one_in_every_context():
    import torch
    from paper_2410_11305_amd import binding as B
    torch.zeros(1, device="cuda")
    side, other, seen = torch.cuda.Stream(), torch.cuda.Stream(), []
    assert B._stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        def in_thread():                       # a thread starts on the default stream, whatever its parent has set
            seen.append(B._stream() == torch.cuda.default_stream().cuda_stream)
            with torch.cuda.stream(other):
                seen.append(B._stream() == other.cuda_stream)
        t = threading.Thread(target=in_thread)
        t.start()
        t.join()
        assert B._stream() == side.cuda_stream
    assert seen == [True, True]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        assert B._stream() == torch.cuda.current_stream().cuda_stream
        torch.zeros(1, device="cuda")
