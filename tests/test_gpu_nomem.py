"""Handles whose device memory runs out in the middle of a call: the call fails,
and the handle goes on from the mesh it holds."""
import numpy as np
import pytest

from paper_1505_04694_amd import inputs, pmesh, pmesh3
from oracle.orc import OracleMesh
from tests.parity import both, compare_mesh, compare_quality, compare_stats
from tests.test_gpu_batch import compare_one

pytestmark = pytest.mark.gpu


class Refusing:
    """Blocks of torch's allocator; the n-th request from arm(n) on is refused, and
    every one of more than `largest` bytes."""

    def __init__(self, largest=1 << 62):
        inner = pmesh.torch_allocator()
        self.left, self.live = -1, {}

        def alloc(nbytes, stream, user):
            self.left -= 1
            if self.left == 0 or nbytes > largest:
                return None
            p = inner.alloc(nbytes, stream, user)
            self.live[p] = nbytes
            return p

        def release(p, nbytes, stream, user):
            assert self.live.pop(p) == nbytes
            inner.release(p, nbytes, stream, user)

        self.inner = inner
        self.of = pmesh.Allocator(pmesh.ALLOC_FN(alloc), pmesh.RELEASE_FN(release), None)

    def arm(self, n):
        self.left = n


@pytest.mark.parametrize("headroom", [1.0, 3.0])
@pytest.mark.parametrize("make", [lambda: inputs.config2(33), lambda: inputs.refine_start(9, 4.0)],
                         ids=["coarsens", "refines"])
@pytest.mark.parametrize("cycle", [("coarsen", "refine"), ("coarsen", "refine", "swap", "smooth")])
def test_refused_allocations_leave_a_handle_that_goes_on(make, headroom, cycle):
    """Every allocation of a cycle refused in turn, each on a fresh handle: what it
    holds then is a mesh on which it and the oracle do the same from there."""
    mi, refused = make(), 0
    phases = ("coarsen", "refine", "swap", "smooth")
    for n in range(1, 200):
        a = Refusing()
        gm = pmesh.Mesh.from_input(mi, seed=2, slack=1.0, pool_headroom=headroom, allocator=a.of)
        a.arm(n)
        failed = None
        for name in cycle:
            try:
                getattr(gm, name)()
            except pmesh.PMError as e:
                assert e.status == pmesh.PM_E_NOMEM, f"request {n}, {name}: {e}"
                failed = name
                break
        a.arm(-1)
        if failed is None:
            gm.close()
            assert not a.live
            break
        refused += 1
        # (renumbered, where the phase left dead slots)
        gm.coarsen(max_rounds=0)
        e = gm.export()
        assert e["valive"].all() and e["talive"].all()
        om, _ = both(type(mi)(xy=e["xy"], tri=e["tri"], metric=e["metric"], tags=e["tags"]), 2)
        compare_mesh(om, gm, f"request {n}, {failed}")
        compare_quality(om, gm, f"request {n}, {failed}")
        for name in phases:
            compare_stats(getattr(om, name)(), getattr(gm, name)(), f"request {n}, {failed}, then {name}")
        compare_mesh(om, gm, f"request {n}, {failed}, end")
        gm.close()
        assert not a.live, f"request {n}, {failed}: blocks not given back"
    assert failed is None and refused > 5


def test_refused_allocations_of_a_creation_are_all_given_back():
    mi, batch, refused = inputs.config2(17), [inputs.make_mesh(k, jitter_seed=k) for k in (9, 5, 7)], 0
    for make in (lambda a: pmesh.Mesh.from_input(mi, allocator=a), lambda a: pmesh.Batch.from_inputs(batch, allocator=a)):
        for n in range(1, 60):
            a = Refusing()
            a.arm(n)
            try:
                make(a.of).close()
            except pmesh.PMError as e:
                assert e.status == pmesh.PM_E_NOMEM, f"request {n}: {e}"
                refused += 1
            assert not a.live, f"request {n}: blocks not given back"
            if a.left > 0:
                break
    assert refused > 20


def test_refused_allocations_in_a_batch():
    """The same with three meshes, which outgrow their ranges and are laid out again."""
    mis, refused = [inputs.refine_start(k, 4.0) for k in (9, 4, 6)], 0
    phases = ("coarsen", "refine", "swap", "smooth")
    for n in range(1, 200):
        a = Refusing()
        b = pmesh.Batch.from_inputs(mis, seed=2, allocator=a.of)
        a.arm(n)
        failed = None
        for name in phases:
            try:
                getattr(b, name)()
            except pmesh.PMError as e:
                assert e.status == pmesh.PM_E_NOMEM, f"request {n}, {name}: {e}"
                failed = name
                break
        a.arm(-1)
        if failed:
            refused += 1
            b.coarsen(max_rounds=0)
            es = [b.export_mesh(i) for i in range(3)]
            oms = [OracleMesh(e["xy"], e["tri"], e["metric"], e["tags"], seed=2) for e in es]
            for name in phases:
                getattr(b, name)()
                for i, om in enumerate(oms):
                    getattr(om, name)()
                    compare_one(om.export(), b.export_mesh(i), f"request {n}, {failed}, then {name}, mesh {i}")
        b.close()
        assert not a.live, f"request {n}, {failed}: blocks not given back"
        if failed is None:
            break
    assert failed is None and refused > 20


def test_tetrahedra_whose_rows_do_not_fit_keep_their_mesh():
    """A refinement to more tetrahedra than the pools' 2^31 entries hold at the
    largest headroom: it fails, calls that need rows fail after it, and the mesh
    that it made is there to export."""
    n = 73
    xyz, tet = inputs.cube_grid(n)
    met = np.tile([1.0, 0.0, 0.0, 1.0, 0.0, 1.0], (len(xyz), 1))
    met[xyz[:, 0] < 0.12] *= 4.0
    m = pmesh3.Mesh3(xyz, tet, met, inputs.unit_cube_tags(xyz), seed=1, pool_headroom=64.0)
    L_up2 = 3.5 / (n - 1) ** 2  # every edge in the dense part, none in the rest
    for call in (lambda: m.refine(L_up2), lambda: m.coarsen(0), lambda: m.smooth(), m.rows, m.colour):
        with pytest.raises(pmesh.PMError) as e:
            call()
        assert e.value.status == pmesh.PM_E_NOMEM
    V, T = m.sizes()
    assert 3 * 65 * 4 * T > 2 ** 31 and V > len(xyz)
    g = m.export()
    assert g["talive"].all() and g["tet"].max() == V - 1
    p = g["xyz"][g["tet"]]
    d = p[:, 1:] - p[:, :1]
    vol = (d[:, 0] * np.cross(d[:, 1], d[:, 2])).sum(1) / 6.0
    assert vol.min() > 0.0 and abs(vol.sum() - 1.0) < 1e-9
    assert np.isfinite(m.quality()[0])
    m.close()


def test_pools_without_memory_for_their_bound_take_the_rows_size():
    """The pools of a small mesh have room for a bound on the rows' entries, about twice
    as many; memory for the headroom times the entries themselves is enough."""
    mi = inputs.make_mesh(33)
    ref = pmesh.Mesh.from_input(mi)
    bound = 4 * (3 * (9 * mi.T + 9 * mi.V) + 4096)  # slack 2: 3 T (1 + 2) + V (2 + 7) entries
    for largest, fits in ((bound, True), (bound * 3 // 4, True), (bound // 4, False)):
        a = Refusing(largest)
        if not fits:
            with pytest.raises(pmesh.PMError) as e:
                pmesh.Mesh.from_input(mi, allocator=a.of)
            assert e.value.status == pmesh.PM_E_NOMEM
        else:
            m = pmesh.Mesh.from_input(mi, allocator=a.of)
            assert (max(a.live.values()) > bound * 9 // 10) == (largest == bound)
            for x, y in zip(m.rows(), ref.rows()):
                assert np.array_equal(x, y)
            assert m.quality() == ref.quality()
            m.close()
        assert not a.live
