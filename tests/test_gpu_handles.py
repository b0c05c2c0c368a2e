"""Host paths of a handle: a coarsening that removes nothing, new coordinates
and metrics taking the place of the old ones, and handles of several threads
and streams polling their read-backs at once."""
import threading

import numpy as np
import pytest

from paper_1505_04694_amd import inputs, pmesh
from tests.parity import both, compare_mesh, compare_stats, run_sweeps

pytestmark = pytest.mark.gpu


def test_coarsening_that_removes_nothing_keeps_mesh_and_rows():
    om, gm = both(inputs.make_mesh(33, layers=2, jitter_seed=1), 1)
    for s in range(3):  # from the second on (nearly) nothing is left to collapse
        compare_stats(om.coarsen(s), gm.coarsen(s), f"coarsen {s}")
        compare_mesh(om, gm, f"coarsen {s}")
    om.refine(), gm.refine()
    run_sweeps(om, gm, 1)


@pytest.mark.parametrize("n", [9, 65])
def test_updates_between_phases(n):
    mi = inputs.make_mesh(n, layers=2, jitter_seed=3)
    _, gm = both(mi, 2)
    gm.coarsen()
    gm.refine()
    e = gm.export()
    inner = e["tags"] == 0
    rng = np.random.default_rng(0)
    for k in range(3):
        met = e["metric"] * rng.uniform(0.5, 1.5)
        xy = e["xy"].copy()
        if k == 1:
            gm.update(metric=met)
        else:
            xy[inner] += rng.uniform(-1e-9, 1e-9, xy[inner].shape)
            gm.update(xy=xy, metric=met if k else None)
            met = met if k else e["metric"]
        g = gm.export()
        assert np.array_equal(g["xy"], xy if k != 1 else e["xy"]) and np.array_equal(g["metric"], met)
        bad = g["xy"].copy()
        bad[:] = bad[::-1]  # every element turned over
        with pytest.raises(pmesh.PMError):
            gm.update(xy=bad, metric=-g["metric"])
        h = gm.export()
        assert np.array_equal(h["xy"], g["xy"]) and np.array_equal(h["metric"], g["metric"])
        e = h
    fresh = type(mi)(xy=e["xy"], tri=e["tri"], metric=e["metric"], tags=e["tags"])
    om, ref = both(fresh, 2)
    gm.set_context(ref.get_context())
    for a in (om, gm):
        a.swap(), a.smooth(kind=1), a.coarsen()
    compare_mesh(om, gm, "after updates")


def test_threads_with_streams_of_their_own():
    import torch
    mis = [inputs.make_mesh(n, layers=2, jitter_seed=n) for n in (17, 33, 65, 97)]
    want = []
    for i, mi in enumerate(mis):
        gm = pmesh.Mesh.from_input(mi, seed=i)
        gm.adapt(max_iterations=2)
        want.append(gm.export())
    got, errs = [None] * len(mis), []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(3):
                    gm = pmesh.Mesh.from_input(mis[i], seed=i)
                    gm.adapt(max_iterations=2)
                    got[i] = gm.export()
                    gm.close()
        except Exception as e:  # noqa: BLE001
            errs.append(e)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(mis))]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not errs, errs
    for a, b in zip(want, got):
        assert all(np.array_equal(a[k], b[k]) for k in ("xy", "tri", "metric", "tags"))
