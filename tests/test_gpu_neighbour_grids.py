"""Neighbour lists of clouds whose grids are at their limits, and what follows the order of their cells."""
import numpy as np
import pytest

import oracle
from paper_2405_13165_amd import workloads as W

pytestmark = pytest.mark.gpu


def check(d, cross=False, n_rows=None):
    from paper_2405_13165_amd import gfdm as g
    ctx = g.Context(0)
    nb = g.build_neighbours(ctx, g.Particles.from_dict(ctx, d), cross_model=cross, n_rows=n_rows)
    rp, col = (t.cpu().numpy() for t in nb.export())
    rp_o, col_o = oracle.neighbours(d, cross=cross) if n_rows is None else oracle.neighbours_rows(d, n_rows, cross=cross)
    assert np.array_equal(rp, rp_o)
    assert np.array_equal(col, col_o)


def pairs_at_faces(origin):
    """Pairs one support apart along a line so sparse that its cells are 57 supports wide: the one just below the upper
    face of a cell, the other alone in the next block of eight cells.  Positions are multiples of 2^-9."""
    h = 514.0 / 512.0
    edge = h * (1.0 + 1e-9)
    for _ in range(10):
        edge *= 1.5
    k = np.arange(1, 7500)
    top = np.floor(8 * k * edge * 512) / 512   # at or below the face between cells 8 k - 1 and 8 k
    x = np.concatenate([[0.0], top, top + h]) + origin
    z = np.zeros(x.size)
    return W._pack(x, z, z, np.full(x.size, h), z, z)


@pytest.mark.parametrize("origin", [0.0, 2.0 ** 40, -(2.0 ** 43), 2.0 ** 43])
def test_far_from_the_origin(origin):
    """Coordinates large against the supports (2^43: positions known to 2e-3 supports)."""
    check(pairs_at_faces(origin))
