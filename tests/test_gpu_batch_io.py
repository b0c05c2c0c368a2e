"""Batches in and out at the edges of the staging blocks: meshes of a few hundred
bytes to several megabytes, given and derived tags, and the mesh an error names."""
import numpy as np
import pytest

from paper_1505_04694_amd import inputs, pmesh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(2,), (3, 2, 2), (17, 160, 5, 161), (150, 230, 2, 90), (400,)])
@pytest.mark.parametrize("tagged", [True, False])
def test_round_trip(sizes, tagged):
    mis = [inputs.make_mesh(n, jitter_seed=k) for k, n in enumerate(sizes)]
    b = pmesh.Batch([(mi.xy, mi.tri, mi.metric, mi.tags if tagged else None) for mi in mis], seed=1)
    for i, mi in enumerate(mis):
        e = b.export_mesh(i)
        assert np.array_equal(e["xy"], mi.xy) and np.array_equal(e["metric"], mi.metric)
        x, y = mi.xy.T
        derived = (x == 0) * 1 + (x == 1) * 2 + (y == 0) * 4 + (y == 1) * 8
        assert np.array_equal(e["tags"], mi.tags if tagged else derived)
        lead = mi.tri.argmin(1)
        assert np.array_equal(e["tri"], np.stack([mi.tri[np.arange(len(lead)), (lead + k) % 3] for k in range(3)], 1))
        assert e["valive"].all() and e["talive"].all()
    b.close()


def test_error_names_the_first_bad_mesh():
    mis = [inputs.make_mesh(n, jitter_seed=n) for n in (5, 9, 6, 7)]
    for i in (1, 3):
        mis[i].tri[-1, 2] = mis[i].V if i == 1 else -1
    with pytest.raises(pmesh.PMError, match="mesh 1: element id out of range"):
        pmesh.Batch([(mi.xy, mi.tri, mi.metric, mi.tags) for mi in mis])


@pytest.mark.parametrize("quality", [pmesh.PM_QUALITY_MEAN_RATIO, pmesh.PM_QUALITY_VASILEVSKII])
def test_batch_of_one_grows_past_its_first_size(quality):
    """One mesh in a batch, refined to many times its slots before and after a
    renumbering, is the mesh that a handle of its own gives."""
    mi = inputs.refine_start()
    b = pmesh.Batch.from_inputs([mi], seed=3, quality=quality)
    m = pmesh.Mesh.from_input(mi, seed=3, quality=quality)

    def same(where):
        e, g = m.export(), b.export_mesh(0)
        assert pmesh.pm_batch_sizes(b.h, 0) == m.sizes() == b.sizes(), where
        for k in ("xy", "tri", "metric", "tags", "valive", "talive"):
            assert np.array_equal(e[k], g[k]), f"{where}: {k}"

    same("create")
    for k in range(3):
        for name in ("refine", "swap", "coarsen", "smooth"):
            kw = dict(max_passes=2) if name == "refine" else dict(sweep=k)
            sm, sb = getattr(m, name)(**kw), getattr(b, name)(**kw)
            assert {k: v for k, v in sm.items() if k != "jp_iterations"} == \
                {k: v for k, v in sb.items() if k != "jp_iterations"}, f"sweep {k} {name}"
            same(f"sweep {k} {name}")
    assert m.sizes()[0] > 4 * mi.V
    (Q, qmin), (Qb, qb) = m.quality(), b.quality_per_mesh()
    assert abs(Q - Qb[0]) <= 1e-12 * abs(Q) and qmin == qb[0]
