"""Calls without a stream run on torch's current one, as it is at each call, in every thread."""
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu


def test_calls_without_a_stream_follow_the_current_one():
    from paper_2601_22101_amd import binding as eco
    seen = {}

    def look(name):
        seen[name] = (eco._stream(None), torch.cuda.current_stream().cuda_stream or None)
        with torch.cuda.stream(torch.cuda.Stream()):
            seen[name + " inner"] = (eco._stream(None), torch.cuda.current_stream().cuda_stream or None)

    for name in ("first", "second"):
        look(name)
        t = threading.Thread(target=look, args=(name + " thread",))
        t.start()
        t.join()
    assert len(seen) == 8 and all(a == b for a, b in seen.values()), seen
    assert seen["first inner"][0] is not None
    # and the call itself: captured work must be on the capturing stream
    x, out = torch.full((4096,), 0x38, dtype=torch.uint8, device="cuda"), torch.zeros(4096, device="cuda")
    s = torch.ones(32, device="cuda")
    eco.eco_dequantize(x, s, 4096, 0, 128, 0, out)
    torch.cuda.synchronize()
    assert bool((out == 1).all())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        eco.eco_dequantize(x, s, 4096, 0, 128, 0, out)
    for k in (2.0, 3.0):
        s.fill_(k)
        graph.replay()
        torch.cuda.synchronize()
        assert bool((out == k).all())


def test_the_raw_lookup_is_found_and_leaves_the_current_stream_alone():
    from paper_2601_22101_amd import binding as eco
    before = torch.cuda.current_stream()
    assert eco._find_raw_stream(torch) is not None                  # this torch has it: small steps rely on it
    assert torch.cuda.current_stream() == before
    with torch.cuda.stream(torch.cuda.Stream()) as s:
        inner = torch.cuda.current_stream()
        assert eco._find_raw_stream(torch)() == inner.cuda_stream and torch.cuda.current_stream() == inner
    graph, x, out = torch.cuda.CUDAGraph(), torch.full((4096,), 0x38, dtype=torch.uint8, device="cuda"), torch.zeros(4096, device="cuda")
    eco._raw_stream = None                                          # the first call of a process, under capture
    scales = torch.full((32,), 3.0, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        eco.eco_dequantize(x, scales, 4096, 0, 128, 0, out)
    for k in (3.0, 5.0):
        scales.fill_(k)
        graph.replay()
        torch.cuda.synchronize()
        assert bool((out == k).all())
