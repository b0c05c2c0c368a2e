"""Row rebuilds at the edges of their forms: hubs whose adjacency rows hold
about 16 entries (one lane group) and about 64 (a wavefront), absorbed by one
another, collapsed onto and flipped around, every row and element against the
oracle."""
import pytest

from paper_1505_04694_amd import inputs
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
