"""Tetrahedral rows at the edges of their forms: stars of 62 to 260 elements and
neighbours around one edge and around one vertex, built, and rebuilt after
collapses that hand over absorbed rows, against the oracle."""
import numpy as np
import pytest

from paper_1505_04694_amd import inputs
from tests.test_gpu3 import both, compare, compare_stats

pytestmark = pytest.mark.gpu


def fan(n, stacked):
    """A closed ring of n vertices around an axis of stacked + 1 vertices: each of the
    axis' inner vertices has 2 n elements, its ends n, with n + 1 neighbours or n + 2."""
    phi = 2 * np.pi * np.arange(n) / n
    z = np.linspace(-0.4, 0.4, stacked + 1)
    xyz = np.vstack([np.stack([0.5 + 0.5 * np.cos(phi), 0.5 + 0.5 * np.sin(phi), np.full(n, 0.5)], 1),
                     np.stack([np.full(len(z), 0.5), np.full(len(z), 0.5), 0.5 + z], 1)])
    a = np.arange(n)
    tet = np.concatenate([np.stack([a, (a + 1) % n, np.full(n, n + k), np.full(n, n + k + 1)], 1)
                          for k in range(stacked)]).astype(np.int32)
    p = xyz[tet]
    neg = np.linalg.det(p[:, 1:] - p[:, :1]) < 0
    tet[neg] = tet[neg][:, [0, 1, 3, 2]]
    tags = np.zeros(len(xyz), np.uint8)
    met = np.tile([1.0, 0.0, 0.0, 1.0, 0.0, 1.0], (len(xyz), 1))
    return inputs.MeshInput3(xyz=xyz, tet=tet, metric=met, tags=tags)


@pytest.mark.parametrize("n", [31, 32, 33, 62, 63, 64, 65, 127, 128, 129, 255, 256, 257])
@pytest.mark.parametrize("stacked", [1, 2, 5])
def test_rows_of_long_stars(n, stacked):
    mi = fan(n, stacked)
    om, gm = both(mi, 3)
    compare(om, gm, "create")
    # short axis: its vertices collapse onto one another, with all they carry
    compare_stats(om.coarsen(0, 0.05, 0.0, 3), gm.coarsen(0, 0.05, 0.0, 3), "coarsen")
    compare(om, gm, "coarsen")


def test_collapse_to_nothing():
    """One tetrahedron whose collapse leaves three vertices and no element."""
    xyz = np.array([[0.2, 0.2, 0.2], [0.5, 0.2, 0.2], [0.2, 0.5, 0.2], [0.2, 0.2, 0.5]])
    met = np.tile([1.0, 0.0, 0.0, 1.0, 0.0, 1.0], (4, 1))
    om, gm = both(inputs.MeshInput3(xyz=xyz, tet=np.array([[0, 1, 2, 3]], np.int32), metric=met,
                                    tags=np.zeros(4, np.uint8)), 3)
    compare_stats(om.coarsen(0, 0.5, 0.0, 5), gm.coarsen(0, 0.5, 0.0, 5), "coarsen")
    compare(om, gm, "coarsen")
    compare_stats(om.refine(0.01), gm.refine(0.01), "refine")
    compare(om, gm, "refine")
