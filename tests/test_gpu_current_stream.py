"""The stream that a call goes to is torch's current one: the default, one in a ``with`` block, another thread's own
(a thread starts on the default stream) and the one that a graph is captured on."""
import threading

import pytest

pytestmark = pytest.mark.gpu


def test_calls_go_to_the_current_stream():
    import torch
    from paper_2505_23317_amd.cfdetr import Encoder

    def same():
        return Encoder._stream() == torch.cuda.current_stream().cuda_stream

    torch.cuda.init()
    assert same() and Encoder._stream() == 0
    side, seen = torch.cuda.Stream(), []
    with torch.cuda.stream(side):
        assert same() and Encoder._stream() == side.cuda_stream
        other = threading.Thread(target=lambda: seen.extend([same(), Encoder._stream()]))
        other.start()
        other.join()
        assert seen == [True, 0]
    graph, x = torch.cuda.CUDAGraph(), torch.zeros(8, device="cuda")
    with torch.cuda.graph(graph):
        x.add_(1)
        assert same() and Encoder._stream() != 0
    assert same() and Encoder._stream() == 0
