"""Calls without a stream argument run on torch's current stream: the handle is that of the stream in force, per thread and inside
nested stream contexts, and a captured graph holds the call."""
import threading

import pytest
import torch

from paper_2101_08458_amd import unit

pytestmark = pytest.mark.gpu


def test_handle_follows_the_current_stream():
    check = lambda: unit._stream(None) == torch.cuda.current_stream().cuda_stream
    torch.cuda.init()
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    assert check()
    with torch.cuda.stream(a):
        assert check() and unit._stream(None) == a.cuda_stream
        with torch.cuda.stream(b):
            assert check() and unit._stream(None) == b.cuda_stream
            seen = []
            t = threading.Thread(target=lambda: seen.append((unit._stream(None), torch.cuda.current_stream().cuda_stream)))
            t.start()
            t.join()
            assert seen[0][0] == seen[0][1] != b.cuda_stream
        assert unit._stream(None) == a.cuda_stream
    assert unit._stream(a) == a.cuda_stream and unit._stream(7) == 7


def test_captured_call_replays():
    a = torch.randint(-64, 64, (3, 512), device="cuda:0", dtype=torch.int8)
    b = torch.randint(-128, 128, (70, 512), device="cuda:0", dtype=torch.int8)
    c = torch.empty((3, 70), device="cuda:0", dtype=torch.int32)
    ws = torch.empty(max(unit.unit_matmul_workspace(3, 70, 512, 512, 512, unit.UNIT_I8), 256), dtype=torch.uint8, device="cuda:0")
    call = lambda: unit.unit_matmul_i8(3, 70, 512, a, 512, b, 512, c, 70, ws)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for _ in range(3):
        a.random_(-64, 64)
        c.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(c.double(), a.double() @ b.double().t())
