"""Neighbour lists where the search's work division can go wrong: cells with
numbers of particles around its row and candidate batches, several support
levels, ghost rows, and clouds whose grids have few or many cells."""
import numpy as np
import pytest

import oracle
from paper_2405_13165_amd import workloads as W

pytestmark = pytest.mark.gpu


def clumps(per, seed, levels):
    """12 clumps of `per` bulk particles (each well inside one support) on a 3x2x2 grid, neighbours of each other's
    edges, over a film of 12 flat clumps of the same size; supports within 20%, or over a factor of six."""
    rng = np.random.default_rng([per, seed])
    corner = 1.3 * np.stack(np.meshgrid(range(3), range(2), range(2), indexing="ij"), -1).reshape(-1, 1, 3)
    bulk = (corner + 0.6 * rng.random((12, per, 3))).reshape(-1, 3)
    film = (corner + 0.6 * rng.random((12, per, 3))).reshape(-1, 3)
    film[:, 2] = 0.05
    pos = np.concatenate([bulk, film])
    pos = pos[rng.permutation(len(pos))]
    n = len(pos)
    model = (pos[:, 2] == 0.05).astype(np.int8)
    h = rng.uniform(0.17, 1.0, n) if levels else rng.uniform(0.8, 1.0, n)
    z = np.zeros(n)
    return W._pack(pos[:, 0], pos[:, 1], pos[:, 2], h, model, np.where(model == 1, W.WALL, W.INTERIOR), z, z, model * 1.0)


def check(d, cross=False, n_rows=None):
    from paper_2405_13165_amd import gfdm as g
    ctx = g.Context(0)
    nb = g.build_neighbours(ctx, g.Particles.from_dict(ctx, d), cross_model=cross, n_rows=n_rows)
    rp, col = (t.cpu().numpy() for t in nb.export())
    rp_o, col_o = oracle.neighbours(d, cross=cross) if n_rows is None else oracle.neighbours_rows(d, n_rows, cross=cross)
    assert np.array_equal(rp, rp_o)
    assert np.array_equal(col, col_o)


@pytest.mark.parametrize("levels", [False, True])
@pytest.mark.parametrize("per", [1, 4, 23, 24, 25, 32, 49, 63, 64, 65, 97])
def test_clumped_cells(per, levels):
    check(clumps(per, 1, levels))


@pytest.mark.parametrize("per,cut", [(5, 1), (24, 300), (33, 500)])
def test_ghost_rows_and_cross_model(per, cut):
    d = clumps(per, 2, True)
    check(d, cross=True)
    check(d, n_rows=len(d["x"]) - min(cut, len(d["x"]) - 1))


@pytest.mark.parametrize("n", [1, 2, 63, 65, 700])
def test_chain(n):
    """A line of particles: a grid one cell thick, far longer than its rows reach."""
    rng = np.random.default_rng(n)
    x = np.cumsum(rng.uniform(0.1, 0.9, n))
    z = np.zeros(n)
    check(W._pack(x, z, z, np.full(n, 1.0), z, z))


@pytest.mark.parametrize("per", [5, 24, 200])
def test_two_far_clumps(per):
    """A bounding box far larger than the supports: cells much wider than the reach of a row, holding up to 60, 288
    and 2,400 particles (each in-cell order has its own kernel)."""
    d = clumps(per, 3, False)
    d["x"] = np.where(np.arange(len(d["x"])) % 2 == 0, d["x"], d["x"] + 1e5)
    check(d)


def test_memory_of_freed_handles():
    """Handles of different sizes built and freed in turn share the context's kept memory; a handle may outlive its
    context."""
    from paper_2405_13165_amd import gfdm as g
    ctx = g.Context(0)
    last = None
    for k, per in enumerate([65, 24, 97, 4, 97]):
        d = clumps(per, 10 + k, False)
        nb = g.build_neighbours(ctx, g.Particles.from_dict(ctx, d))
        rp, col = (t.cpu().numpy() for t in nb.export())
        rp_o, col_o = oracle.neighbours(d)
        assert np.array_equal(rp, rp_o) and np.array_equal(col, col_o)
        if k % 2:
            nb.close()
        else:
            last = nb  # frees the one before it
    ctx.close()
    last.close()
