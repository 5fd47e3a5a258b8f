"""Reading the status words of a stream under capture is refused, and leaves nothing in the graph:
what was captured around the refused call replays as what was launched eagerly."""
import ctypes as ct

import pytest

import workloads as wl
from tests.test_gpu_parity import dev, say

pytestmark = pytest.mark.gpu


def test_refused_and_nothing_recorded():
    import torch

    import paper_2510_05814_amd as smoe
    say("status under capture")
    W, H = 200, 120
    m = dev(wl.random_model(300, 3, 1, W, H, 3))
    grid = smoe.make_grid(W, H)
    want = smoe.bin(m, 3, 1, grid)
    P = want.read_status()[1][0]
    b = smoe.Bins(300, 3, 1, smoe.tiles(W, H), P, render_only=True)
    hip = ct.CDLL("libamdhip64.so.7")
    nodes = []
    for ask in (False, True):
        g = torch.cuda.CUDAGraph(keep_graph=True)
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            g.capture_begin()
            smoe.bin(m, 3, 1, grid, bins=b, grow=False)
            if ask:
                with pytest.raises(RuntimeError):
                    b.read_status()
            g.capture_end()
        n = ct.c_size_t()
        assert hip.hipGraphGetNodes(ct.c_void_p(g.raw_cuda_graph()), None, ct.byref(n)) == 0
        nodes.append(n.value)
    assert nodes[0] == nodes[1] > 0
    for _ in range(3):
        b.ws.fill_(0xFF)
        g.replay()
        torch.cuda.synchronize()
        assert b.read_status()[1] == want.read_status()[1]
        assert torch.equal(b.vals(P), want.vals(P)) and torch.equal(b.keys(P), want.keys(P))
