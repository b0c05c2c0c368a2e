"""Tetrahedral colourings at the edges of their forms (one thread a vertex, two,
iterations with a one-block end) and of a vertex with more neighbours before it
than a record holds, against the oracle's greedy one."""
import numpy as np
import pytest

from paper_1505_04694_amd import inputs
from tests.test_gpu3 import both

pytestmark = pytest.mark.gpu


def check(mi, sizes, seed, ctxs=1):
    om, gm = both(mi, seed)
    rng = np.random.default_rng(seed)
    for n in sizes:
        active = np.zeros(mi.V, np.uint8)
        active[rng.permutation(mi.V)[:n]] = 1
        for ctx in range(ctxs):
            co, no = om.colour(active, ctx)
            cg, ng = gm.colour(active, ctx)
            assert no == ng and np.array_equal(co, cg), f"{n} of {mi.V} vertices, context {ctx}"


@pytest.mark.parametrize("sizes", [(0, 1, 64, 1023, 1024, 1025), (2047, 2048, 2049, 4913)])
def test_colour_list_lengths(sizes):
    check(inputs.make_mesh3(17, jitter_seed=1), sizes, 5)


def star(k):
    """The cube's surface, k x k vertices a face, joined to its centre."""
    xyz, tet = inputs.cube_grid(k)
    outer = np.flatnonzero(inputs.unit_cube_tags(xyz))
    place = np.full(len(xyz), -1)
    place[outer] = np.arange(len(outer))
    tri = np.concatenate([tet[:, f] for f in ([1, 2, 3], [0, 3, 2], [0, 1, 3], [0, 2, 1])])
    c = xyz[tri]
    flat = [np.any([(np.abs(c[:, :, a] - x) < 1e-12).all(1) for a in range(3) for x in (0.0, 1.0)], axis=0)][0]
    tri = place[tri[flat]]
    pts = np.vstack([xyz[outer], [[0.5, 0.5, 0.5]]])
    t = np.hstack([np.full((len(tri), 1), len(outer)), tri]).astype(np.int32)
    p = pts[t]
    neg = np.linalg.det(p[:, 1:] - p[:, :1]) < 0
    t[neg] = t[neg][:, [0, 1, 3, 2]]
    met = np.tile([1.0, 0.0, 0.0, 1.0, 0.0, 1.0], (len(pts), 1))
    return inputs.MeshInput3(xyz=pts, tet=t, metric=met, tags=inputs.unit_cube_tags(pts))


@pytest.mark.parametrize("k", [3, 4, 5, 9, 25])
def test_colour_high_degree(k):
    mi = star(k)  # the centre has 26, 56, 98, 386 and 3458 neighbours
    check(mi, (mi.V,), 7, ctxs=6)
