"""Device memory of the neighbour handles: when it is handed on, to whom, and what happens under stream capture."""
import threading

import numpy as np
import pytest

from paper_2405_13165_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def built(ctx, d):
    from paper_2405_13165_amd import gfdm as g
    p = g.Particles.from_dict(ctx, d)
    return p, g.build_neighbours(ctx, p)


@pytest.mark.parametrize("mode", ["relaxed", "thread_local"])
def test_handle_freed_during_a_capture(mode):
    """Freeing a handle leaves a capture alone where hipFree does: a relaxed one, and another thread's."""
    from paper_2405_13165_amd import gfdm as g
    ctx = g.Context(0)
    _, nb = built(ctx, W.plain_cube(9))
    a = torch.zeros(8, device=ctx.device)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, capture_error_mode=mode):
        a.add_(1)
        if mode == "relaxed":
            nb.close()
        else:
            t = threading.Thread(target=nb.close)
            t.start()
            t.join()
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert a[0].item() == k + 1
