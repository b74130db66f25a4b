"""The counters of the QR fallback's queue, one cleared by the call before: eager calls one after another, with graph replays,
the autotuner and calls that queue nothing between them, all queue exactly the rows whose condition exceeds the limit."""
import pytest
import torch

from paper_2405_13165_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_queue_counts_over_calls():
    from paper_2405_13165_amd import gfdm as g
    ctx = g.Context(0)
    d = W.mixed_block_film(factor=4)
    p = g.Particles.from_dict(ctx, d)
    nb = g.build_neighbours(ctx, p)
    u = torch.as_tensor(W.test_field(d["x"], d["y"], d["z"])[0], device=ctx.device).clone()
    kappa = torch.empty(p.n, dtype=torch.float32, device=ctx.device)
    g.gfdm_weights(ctx, p, nb, kappa=kappa)
    some, none = g.ls_params(kappa_max=float(kappa.median())), g.ls_params()
    w = torch.empty((nb.nnz, 4), dtype=torch.float32, device=ctx.device)
    y = torch.empty((4, p.n), dtype=torch.float64, device=ctx.device)

    status = torch.empty(p.n, dtype=torch.int8, device=ctx.device)

    def eager(prm):
        a = w.zero_().clone(), y.zero_().clone()
        status.fill_(-1)
        g.gfdm_weights_apply(ctx, p, nb, u, 0xF, g.GF_F32, params=prm, w_out=a[0], out=a[1], status=status)
        assert torch.equal(status, (kappa > prm.kappa_max).to(torch.int8))   # 1: by the QR, 0: not
        return a

    def same(a, b):
        return torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])

    ref_some, ref_none = eager(some), eager(none)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        g.gfdm_weights_apply(ctx, p, nb, u, 0xF, g.GF_F32, params=some, w_out=w, out=y)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.gfdm_weights_apply(ctx, p, nb, u, 0xF, g.GF_F32, params=some, w_out=w, out=y)
    torch.cuda.synchronize()
    for k in range(6):
        assert same(eager(some), ref_some), k
        if k % 3 == 1:
            assert same(eager(none), ref_none), k
        if k % 2:
            w.zero_()
            y.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert same((w, y), ref_some), k
        if k == 3:
            teams = g.set_team_sizes(ctx)
            g.autotune(ctx, p, nb)
            g.set_team_sizes(ctx, teams["weights"], teams["apply"], teams["fused"])
    _, st = g.gfdm_weights(ctx, p, nb, params=some, stats=True)
    assert 0.4 * p.n < st["n_fallback"] < 0.6 * p.n
    _, st = g.gfdm_weights(ctx, p, nb, params=none, stats=True)
    assert st["n_fallback"] == 0
