"""The pressure solve where its packed tiles and folded reductions can go wrong: tiles with one row or a few, groups of
very different row lengths, rows beyond the tiles, matrices with and without a staged vector, small and large updates."""
import numpy as np
import pytest
import torch

from paper_2405_13165_amd import workloads as W

pytestmark = pytest.mark.gpu


def system(kind, size):
    rng = np.random.default_rng([31, size])
    if kind == "film":
        i, j = (a.ravel() for a in np.meshgrid(np.arange(size), np.arange(7), indexing="ij"))
        x, y = i + rng.uniform(-0.2, 0.2, i.size), j + rng.uniform(-0.2, 0.2, i.size)
        z = np.zeros(i.size)
        return W._pack(x, y, z, np.full(i.size, 3.0), np.ones(i.size), np.full(i.size, W.WALL), z, z, z + 1)
    x, y, z = W.jittered_cube(size, 1.0, rng)
    n = x.size
    h = np.full(n, 3.0)
    if kind == "uneven":  # rows of about 20 to more than 128 entries
        h = np.where(x < size / 2, 2.6, 3.9)
    return W._pack(x, y, z, h, np.zeros(n), np.zeros(n))


@pytest.mark.parametrize("mixed", [0, 1, 2])
@pytest.mark.parametrize("kind,size,cap", [("film", 5, 0), ("film", 37, 0), ("film", 37, 8), ("cube", 4, 0), ("cube", 13, 0),
                                           ("cube", 13, 64), ("uneven", 14, 0), ("cube", 52, 0)])
def test_implicit_step(kind, size, cap, mixed):
    """(I - a Lap) p = b against the residual and, on small systems, the dense solution in numpy (rtol 1e-11; FP64 matrix,
    condition number a few tens, so the solution's relative error stays below 1e-9)."""
    from paper_2405_13165_amd import gfdm as g
    d = system(kind, size)
    n = d["x"].size
    ctx = g.Context(0)
    ctx.set_tile_capacity(cap)
    p = g.Particles.from_dict(ctx, d)
    nb = g.build_neighbours(ctx, p)
    if kind == "uneven":
        assert nb.max_row > 128
    w = g.gfdm_weights(ctx, p, nb, g.GF_BATCHED, g.GF_F64)
    rng = np.random.default_rng(n)
    a = 0.3
    rt = np.full(n, g.ROW_IMPLICIT, np.int8)
    rt[:: 7] = g.ROW_DIRICHLET
    b = torch.as_tensor(rng.standard_normal(n), device=ctx.device)
    x, st = g.poisson_solve(ctx, p, nb, w, rt, b, params=g.solve_params(rtol=1e-11, mixed=mixed, implicit_a=a))
    assert st["converged"]
    rp, col = (t.cpu().numpy() for t in nb.export())
    row = np.repeat(np.arange(n), np.diff(rp))
    lap = w[:, 3].cpu().numpy()
    val = np.where(rt[row] == g.ROW_DIRICHLET, (row == col) * 1.0, (row == col) - a * lap)
    xs, bs = x.cpu().numpy(), b.cpu().numpy()
    r = bs - np.bincount(row, val * xs[col], n)
    assert np.linalg.norm(r) <= 1.1e-11 * np.linalg.norm(bs)
    if n <= 2500:
        A = np.zeros((n, n))
        A[row, col] = val
        ref = np.linalg.solve(A, bs)
        assert np.linalg.norm(xs - ref) <= 1e-9 * np.linalg.norm(ref)
    # a second solve from the solution: nothing to do
    x2, st2 = g.poisson_solve(ctx, p, nb, w, rt, b, x0=x, params=g.solve_params(rtol=2e-11, mixed=mixed, implicit_a=a))
    assert st2["inner_its_total"] == 0 and torch.equal(x, x2)
