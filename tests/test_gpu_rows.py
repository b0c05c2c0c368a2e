"""Row rebuilds at the edges of their forms: hubs whose adjacency rows hold
about 16 entries (one lane group) and about 64 (a wavefront), absorbed by one
another, collapsed onto and flipped around, every row and element against the
oracle."""
import numpy as np
import pytest

from paper_1505_04694_amd import inputs, pmesh
from tests.parity import both, compare_mesh, compare_stats

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("hubs,layers", [(1, 2), (2, -1), (2, 2)])
@pytest.mark.parametrize("ring", [14, 15, 16, 17, 18, 32, 34, 62, 63, 64, 65, 66, 68])
def test_hub_rows(ring, hubs, layers, order):
    mi = inputs.fan(ring, hubs=hubs, layers=layers)
    om, gm = both(mi, 3, tune=dict(commit_order=order, small_work=1))
    for name in ("swap", "coarsen"):
        compare_stats(getattr(om, name)(0), getattr(gm, name)(0), f"{name} ring={ring}")
        compare_mesh(om, gm, f"{name} ring={ring} hubs={hubs}")


def spiral(m):
    """A fan that winds past a full turn around vertex 0, whose overlapping sheet
    flips an edge of vertex 0 onto vertex 2, a neighbour of it already: two of its
    elements then go from vertex 0 to vertex 2."""
    def at(r, deg):
        return r * np.cos(np.deg2rad(deg)), r * np.sin(np.deg2rad(deg))
    ring = [0.0, 60.0] + list(np.linspace(120, 300, m))
    k = len(ring)
    xy = [(0.0, 0.0)] + [at(1, a) for a in ring] + [at(0.5, 0), at(0.5, 120), (1.5, 1.0), (0.3, 1.6)]
    s1, s2, y, y2 = k + 1, k + 2, k + 3, k + 4
    tri = [(0, i, i + 1) for i in range(1, k)] + [(0, k, s1), (0, s1, s2), (s2, s1, 2), (2, 1, y), (2, y, y2), (2, y2, s2)]
    return np.array(xy), np.array(tri, np.int32)


@pytest.mark.parametrize("tune", [dict(), dict(commit_order=1, small_work=1), dict(commit_order=2, small_work=1)])
@pytest.mark.parametrize("m", [4, 9, 12, 13, 14, 40, 60, 61, 62, 70])
def test_rows_of_an_edge_that_comes_twice(m, tune):
    xy, tri = spiral(m)
    g = pmesh.Mesh(xy, tri, np.tile([1.0, 0.0, 1.0], (len(xy), 1)), np.zeros(len(xy), np.uint8), tune=tune)
    g.swap(max_rounds=1)
    e = g.export()
    t = e["tri"]
    edges = [(a, b) for x in t.tolist() for a, b in ((x[0], x[1]), (x[1], x[2]), (x[2], x[0]))]
    assert edges.count((0, 2)) == 2
    nn_off, nn, ne_off, ne = g.rows()
    for v in range(len(xy)):
        rows = np.flatnonzero((t == v).any(1))
        assert np.array_equal(ne[ne_off[v]:ne_off[v + 1]], rows), f"elements of {v}"
        assert np.array_equal(nn[nn_off[v]:nn_off[v + 1]], np.setdiff1d(t[rows], [v])), f"neighbours of {v}"
    g.close()
