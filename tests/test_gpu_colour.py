"""Colourings at the edges of their forms (one launch, one block after a scan
by many, chunks of 256 and of 512 entries with a one-block finish), and rows
with more predecessors than a record holds, against the oracle's greedy one."""
import numpy as np
import pytest

from paper_1505_04694_amd import inputs, pmesh
from tests.parity import both

pytestmark = pytest.mark.gpu


def check(mi, sizes, seed=5):
    om, gm = both(mi, seed)
    rng = np.random.default_rng(seed)
    for ctx, n in enumerate(sizes):
        active = np.zeros(mi.V, np.uint8)
        active[rng.permutation(mi.V)[:n]] = 1
        for k in range(2):  # the second call has the first one's iteration counts
            co, no = om.colour(active, ctx)
            cg, ng = gm.colour(active, ctx)
            assert no == ng and np.array_equal(co, cg), f"{n} of {mi.V} vertices, call {k}"


@pytest.mark.parametrize("sizes", [(0, 1, 2, 64, 511, 512, 513), (1023, 2047, 2048, 2049), (8191, 8192, 8193, 16641)])
def test_colour_list_lengths(sizes):
    check(inputs.make_mesh(129, jitter_seed=2), sizes)


def test_colour_chunk_lengths():
    check(inputs.make_mesh(725), (1 << 19, (1 << 19) + 1, 725 * 725))


@pytest.mark.parametrize("k", [8, 9, 30, 96])
def test_colour_high_degree(k):
    mi = inputs.fan(k, hubs=2, radius=0.3, layers=-1)
    check(mi, (mi.V, mi.V - 5), seed=1)
    check(mi, (mi.V,), seed=4)


def test_iterations_count_the_one_block_finish():
    """A long list's iterations are its launches, and at least one pass in the finish
    that colours what they leave."""
    m = pmesh.Mesh.from_input(inputs.make_mesh(257, jitter_seed=4))
    m.smooth()  # the next call stops iterating where the finish takes over
    m.profile(1 << pmesh.KERNELS.index("jp"))
    st = m.smooth(sweep=1)
    p = m.profile_read(["jp"])["jp"]
    assert p["launches"] > 1 and st["jp_iterations"] >= p["launches"]
    m.close()
