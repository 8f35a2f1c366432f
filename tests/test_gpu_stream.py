"""The binding's default stream is torch's current one: of the device, the thread and the moment of the call."""
import threading

import pytest
import torch

import paper_2604_26666_amd as fact

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["default", "side", "nested", "thread", "capture"])
def test_default_stream_is_the_current_one(where):
    torch.cuda.synchronize()
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    seen = lambda: (fact.binding._stream(None), torch.cuda.current_stream().cuda_stream)
    got = []
    if where == "default":
        got.append(seen() + (0,))
    elif where == "side":
        with torch.cuda.stream(side):
            got.append(seen() + (side.cuda_stream,))
        got.append(seen() + (0,))
    elif where == "nested":
        with torch.cuda.stream(side):
            with torch.cuda.stream(other):
                got.append(seen() + (other.cuda_stream,))
            got.append(seen() + (side.cuda_stream,))
    elif where == "thread":
        with torch.cuda.stream(side):                       # a new thread starts on the default stream
            t = threading.Thread(target=lambda: got.append(seen() + (0,)))
            t.start()
            t.join()
    else:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            got.append(seen() + (side.cuda_stream,))
            torch.zeros(1, device="cuda")
    assert got and all(a == b == c for a, b, c in got), got
