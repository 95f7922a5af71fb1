"""The reading behind isovolumes from vertex components, on the oracle: every isovolume is named by the one of its two
vertex components whose first vertex is larger, and there is one isovolume less than components."""
import itertools

import numpy as np
import pytest
from scipy.sparse import coo_matrix
from scipy.sparse.csgraph import connected_components

from oracle import iso as OI


def vertex_components(above):
    """First vertex of each vertex's component among the Kuhn mesh's edges between vertices on one side."""
    g = np.arange(above.size).reshape(above.shape)
    rows, cols = [], []
    for d in itertools.product((0, 1), repeat=4):
        if any(d):
            lo = tuple(slice(0, n - k) for n, k in zip(above.shape, d))
            hi = tuple(slice(k, None) for k in d)
            same = above[lo] == above[hi]
            rows.append(g[lo][same])
            cols.append(g[hi][same])
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    n, c = connected_components(coo_matrix((np.ones(len(rows)), (rows, cols)), shape=(g.size, g.size)), directed=False)
    first = np.full(n, g.size)
    np.minimum.at(first, c, np.arange(g.size))
    return n, first[c]


@pytest.mark.parametrize("seed", range(12))
def test_isovolumes_are_pairs_of_vertex_components(seed):
    rng = np.random.default_rng(seed)
    shape = tuple(rng.integers(2, 6, size=4))
    f = rng.normal(size=shape) if seed % 2 else rng.choice([-1.0, 0.0, 1.0], size=shape, p=[0.7, 0.1, 0.2])
    f = f.astype(np.float32)
    o = OI.track_iso(f, 0.0)
    n, comp = vertex_components(f >= 0.0)
    assert o.n_components == (n - 1 if o.n_hits else 0)
    nt, nz, ny, nx = shape
    v, M = o.edge_id // 15, o.edge_id % 15 + 1
    w = v + (M & 1) + ((M >> 1) & 1) * nx + ((M >> 2) & 1) * nx * ny + (M >> 3) * nx * ny * nz
    name = np.maximum(comp[v], comp[w])
    for label in np.unique(o.label):
        assert len(np.unique(name[o.label == label])) == 1
    assert len(np.unique(name)) == o.n_components
