"""The framework's work, as a user's program has it done: one case per kind of
call and size, each through the public entry points (pmesh.Mesh, pmesh.Batch,
pmesh3.Mesh3, pmesh.QualityFn and the C ABI's export to device memory).

A case is a dict of plain values; its "kind" says which path it takes:

  adapt    create a handle from device arrays, Algorithm 1 (pm_adapt), export to device arrays
  sweeps   create, coarsen -> refine -> swap -> smooth sweeps, export
  step     create, quality + adjoint, plain and gradient smoothing at full
           size, one sweep, quality, export
  quality  QualityFn forward and backward on a handle the program keeps
  smooth   new coordinates into a kept handle, then smoothing sweeps
  psi      one time step of the psi benchmark: the adapted mesh of the last
           step with the next step's metric, Algorithm 1, export
  batch    many small meshes from host arrays in one handle, sweeps, export
  tet      tetrahedra: create, sweeps without swaps, export
  tetpsi   tetrahedra: psi extruded, coarsen and refine, one smoothing, export

Meshes are the seeded grids and fields of the package's inputs module: jitter,
layer amplitude, width and tangential size (or psi's phase) come from the
seed. "ratio" scales a metric so that its ideal element count is that multiple
of the start's elements: below 1 the mesh mostly coarsens, above 1 it refines.
"""
import math

import numpy as np
import torch

from paper_1505_04694_amd import inputs, pmesh, pmesh3

MEAN, VASI = pmesh.PM_QUALITY_MEAN_RATIO, pmesh.PM_QUALITY_VASILEVSKII
LAPLACE, GRADIENT, MINMAX = pmesh.PM_SMOOTH_LAPLACE, pmesh.PM_SMOOTH_GRADIENT, pmesh.PM_SMOOTH_MINMAX


def listed():
    return [
        # the smallest whole call: a 33 x 33 mesh adapted once, all launch and read-back latency
        dict(name="adapt_33", kind="adapt", n=33, layers=2, ratio=1.0, quality=MEAN),
        # an ordinary mesh near its metric's size, some collapses, splits and flips; the size-aware functional
        dict(name="adapt_257_vasilevskii", kind="adapt", n=257, layers=2, ratio=0.7, quality=VASI),
        # three sweeps on a million vertices under a coarse one-layer metric
        dict(name="sweeps_1025", kind="sweeps", n=1025, layers=1, sweeps=3),
        # the benchmark's step: every phase and the adjoint at 4.2 million vertices, the largest mesh
        dict(name="step_2049", kind="step", n=2049),
        # the functional in an optimisation loop, forward and backward: a small mesh, latency counts
        dict(name="quality_129_vasilevskii", kind="quality", n=129, quality=VASI),
        # the same at full size, bandwidth counts
        dict(name="quality_2049", kind="quality", n=2049, quality=MEAN),
        # ten sweeps of the gradient smoother, as a program that only smooths runs them
        dict(name="smooth_gradient_1025", kind="smooth", n=1025, smoother=GRADIENT, sweeps=10, quality=MEAN),
        # the min-max smoother on a mesh of ordinary size
        dict(name="smooth_minmax_257", kind="smooth", n=257, smoother=MINMAX, sweeps=3, quality=MEAN),
        # the paper's time-varying benchmark: a step at about half a million elements
        dict(name="psi_201", kind="psi", n=201, target=550000),
        # many small meshes at once, from host arrays
        dict(name="batch_64", kind="batch", count=64, nmin=17, nmax=129, sweeps=2),
        # a small tetrahedral mesh, one sweep
        dict(name="tet_11", kind="tet", n=11, ratio=1.0, sweeps=1),
        # the paper's benchmark extruded: 132 thousand tetrahedra at the start
        dict(name="tetpsi_29", kind="tetpsi", n=29, target=210000, iterations=2),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["adapt", "adapt", "sweeps", "step", "quality", "quality", "smooth", "smooth", "psi", "batch",
                       "tet", "tetpsi"])
    if kind == "adapt":
        return dict(kind=kind, n=_logint(rng, 17, 700), layers=rng.choice([1, 2]),
                    ratio=round(math.exp(rng.uniform(math.log(0.1), math.log(2.0))), 3), quality=rng.choice([MEAN, VASI]))
    if kind == "sweeps":
        return dict(kind=kind, n=_logint(rng, 33, 1200), layers=rng.choice([1, 2]), sweeps=rng.choice([1, 2, 3]))
    if kind == "step":
        return dict(kind=kind, n=_logint(rng, 65, 1700))
    if kind == "quality":
        return dict(kind=kind, n=_logint(rng, 17, 2048), quality=rng.choice([MEAN, VASI]))
    if kind == "smooth":
        return dict(kind=kind, n=_logint(rng, 17, 1400), smoother=rng.choice([LAPLACE, GRADIENT, MINMAX]),
                    sweeps=rng.choice([1, 2, 5, 10]), quality=rng.choice([MEAN, VASI]))
    if kind == "psi":
        return dict(kind=kind, n=_logint(rng, 33, 201), target=_logint(rng, 10000, 550000))
    if kind == "batch":
        return dict(kind=kind, count=_logint(rng, 4, 96), nmin=rng.randint(9, 33), nmax=rng.randint(49, 129),
                    sweeps=rng.choice([1, 2]))
    if kind == "tet":
        return dict(kind=kind, n=rng.randint(5, 23), ratio=round(math.exp(rng.uniform(math.log(0.2), math.log(1.5))), 3),
                    sweeps=rng.choice([1, 2]))
    n = rng.randint(11, 27)
    return dict(kind=kind, n=n, target=_logint(rng, 4000, min(150000, 8 * n ** 3)), iterations=rng.choice([1, 2]))


# ---- inputs ---------------------------------------------------------------------

def _field(rng):
    """The batched workload's ranges of the layer field."""
    return dict(amp=float(rng.uniform(0.05, 0.2)), width=float(rng.uniform(0.02, 0.1)), ht=float(rng.uniform(0.05, 0.2)))


def _grid(case, seed, n=None):
    """The seeded grid of a 2D case; the step and the kept handles use the benchmark's two-layer field."""
    rng = np.random.default_rng([seed, 2])
    n = n or case["n"]
    if case["kind"] in ("step", "quality", "smooth"):
        return inputs.make_mesh(n, layers=2, jitter_seed=seed)
    mi = inputs.make_mesh(n, layers=case.get("layers", 1), jitter_seed=seed, **_field(rng))
    if "ratio" in case:
        mi.metric *= case["ratio"] * mi.T / inputs.ideal_elements(mi.xy, mi.tri, mi.metric)
    return mi


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _arrays(mi):
    return (_dev(mi.xy), _dev(mi.tri), _dev(mi.metric), _dev(mi.tags))


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case, seed=seed)
    if kind not in ("quality", "smooth"):
        s["buffers"] = _buffers(case, "cpu" if kind == "batch" else "cuda")
    if kind in ("adapt", "sweeps", "step"):
        s["arrays"] = _arrays(_grid(case, seed))
    elif kind in ("quality", "smooth"):
        # the handle stands on the undisturbed grid; each pass brings its own coordinates
        mi = _grid(case, seed)
        s["xy"], tri, s["metric"], tags = _arrays(mi)
        s["mesh"] = pmesh.Mesh(s["xy"], tri, s["metric"], tags, seed=seed, quality=case["quality"])
        if kind == "quality":
            s["xy"].requires_grad_()
            s["metric"].requires_grad_()
    elif kind == "psi":
        n, ph = case["n"], float(np.random.default_rng([seed, 3]).uniform(0.0, 2.0 * math.pi))
        g = inputs.grid(min(n, 101))
        eps = inputs.psi_eps(*g, case["target"])
        xy, tri = inputs.grid(n)
        m = pmesh.Mesh(_dev(xy), _dev(tri), _dev(inputs.psi_metric(xy, ph, eps)), _dev(inputs.unit_square_tags(xy)), seed=seed)
        m.adapt(max_iterations=2)
        e = m.export()
        m.close()
        met = inputs.psi_metric(e["xy"], ph + 2.0 * math.pi / 50, eps)
        s["arrays"] = (_dev(e["xy"]), _dev(e["tri"]), _dev(met), _dev(e["tags"]))
    elif kind == "batch":
        rng = np.random.default_rng([seed, 4])
        ns = np.exp(rng.uniform(math.log(case["nmin"]), math.log(case["nmax"]), case["count"]))
        mis = [inputs.make_mesh(int(round(k)), jitter_seed=seed + i, **_field(rng)) for i, k in enumerate(ns)]
        for mi in mis:  # between a quarter and all of its elements stay
            mi.metric *= rng.uniform(0.25, 1.0) * mi.T / inputs.ideal_elements(mi.xy, mi.tri, mi.metric)
        s["meshes"] = [(mi.xy, mi.tri, mi.metric, mi.tags) for mi in mis]
    elif kind == "tet":
        rng = np.random.default_rng([seed, 5])
        mi = inputs.make_mesh3(case["n"], jitter_seed=seed, amp_y=float(rng.uniform(0.0, 0.1)), **_field(rng))
        mi.metric *= (case["ratio"] * mi.T / inputs.ideal_elements3(mi.xyz, mi.tet, mi.metric)) ** (2.0 / 3.0)
        s["arrays"] = (_dev(mi.xyz), _dev(mi.tet), _dev(mi.metric), _dev(mi.tags))
    else:
        ph = float(np.random.default_rng([seed, 6]).uniform(0.0, 2.0 * math.pi))
        eps = inputs.psi_start3(min(case["n"], 13), target=case["target"]).info["eps"]
        xyz, tet = inputs.cube_grid(case["n"])
        s["arrays"] = (_dev(xyz), _dev(tet), _dev(inputs.psi_metric3(xyz, ph, eps)), _dev(inputs.unit_cube_tags(xyz)))
    return s


# ---- one pass -------------------------------------------------------------------

def _room(case):
    """Vertices and elements that the program keeps room for in its own arrays:
    what the start holds, and about twice what its metric asks for (tetrahedra
    are never swapped, and bisection leaves many times the ideal count)."""
    kind = case["kind"]
    if kind in ("tet", "tetpsi"):
        T = 6 * (case["n"] - 1) ** 3
        T = int(24 * (max(T, case["target"]) if kind == "tetpsi" else T * max(1.0, case["ratio"]))) + 4096
        return max(T // 4, case["n"] ** 3), T
    if kind == "batch":
        n = case["nmax"]
        return 2 * case["count"] * n * n, 4 * case["count"] * n * n
    T = 2 * (case["n"] - 1) ** 2
    if kind in ("sweeps", "step"):  # the unscaled layer fields ask for some hundred elements
        T = min(T, 32768)
    T = int(2 * max(T, case["target"] if kind == "psi" else T * case.get("ratio", 0.0))) + 4096
    return T, T


def _buffers(case, device):
    """The program's own arrays for the adapted mesh (the part past its sizes stays zero)."""
    V, T = _room(case)
    d = 3 if case["kind"] in ("tet", "tetpsi") else 2
    return dict(xy=torch.zeros((V, d), dtype=torch.float64, device=device),
                metric=torch.zeros((V, d * (d + 1) // 2), dtype=torch.float64, device=device),
                elements=torch.zeros((T, d + 1), dtype=torch.int32, device=device),
                tags=torch.zeros(V, dtype=torch.uint8, device=device))


def _export(m, buf):
    """The mesh into the program's device arrays, through the C ABI, and its sizes."""
    three = isinstance(m, pmesh3.Mesh3)
    V, T = m.sizes()
    if V > len(buf["xy"]) or T > len(buf["elements"]):
        raise ValueError("the program's arrays are too small: %d vertices, %d elements" % (V, T))
    lib = pmesh3.lib() if three else pmesh.lib()
    st = (lib.pm3_mesh_export if three else lib.pm_mesh_export)(
        m.h, buf["xy"].data_ptr(), buf["elements"].data_ptr(), buf["metric"].data_ptr(), buf["tags"].data_ptr(),
        None, None, pmesh.PM_MEM_DEVICE)
    if st != pmesh.PM_OK:
        raise pmesh.PMError(st, "export")
    return dict(buf, V=V, T=T)


def run(state):
    case, seed = state["case"], state["seed"]
    kind = case["kind"]
    if kind == "quality":
        Q = pmesh.QualityFn.apply(state["xy"], state["metric"], state["mesh"])
        gx, gm = torch.autograd.grad(Q, (state["xy"], state["metric"]))
        return dict(Q=Q, gx=gx, gm=gm)
    if kind == "smooth":
        m = state["mesh"]
        m.update(xy=state["xy"])
        m.smooth(kind=case["smoother"], sweeps=case["sweeps"])
        xy = torch.empty_like(state["xy"])
        st = pmesh.lib().pm_mesh_export(m.h, xy.data_ptr(), None, None, None, None, None, pmesh.PM_MEM_DEVICE)
        if st != pmesh.PM_OK:
            raise pmesh.PMError(st, "export")
        return dict(xy=xy)
    if kind == "batch":
        b = pmesh.Batch(state["meshes"], seed=seed)
        for k in range(case["sweeps"]):
            b.sweep(k)
        Q, qmin = b.quality_per_mesh()
        buf, sizes, v, t = state["buffers"], [], 0, 0
        for i in range(b.count()):
            e = b.export_mesh(i)
            V, T = len(e["xy"]), len(e["tri"])
            for k in ("xy", "metric", "tags"):
                buf[k][v:v + V] = torch.from_numpy(e[k])
            buf["elements"][t:t + T] = torch.from_numpy(e["tri"])
            sizes.append((V, T))
            v, t = v + V, t + T
        b.close()
        return dict(buf, Q=Q, qmin=qmin, sizes=np.array(sizes))
    if kind in ("tet", "tetpsi"):
        m = pmesh3.Mesh3(*state["arrays"], seed=seed)
        if kind == "tet":
            for k in range(case["sweeps"]):
                m.sweep(k)
        else:
            for k in range(case["iterations"]):
                m.coarsen(k)
                m.refine()
            m.smooth()
        Q, qmin = m.quality()
        out = dict(_export(m, state["buffers"]), Q=Q, qmin=qmin)
        m.close()
        return out
    m = pmesh.Mesh(*state["arrays"], seed=seed, quality=case.get("quality", MEAN))
    out = {}
    if kind == "adapt":
        m.adapt()
    elif kind == "psi":
        m.adapt(max_iterations=2)
    elif kind == "sweeps":
        for k in range(case["sweeps"]):
            m.sweep(k)
    else:
        out["Q0"], out["qmin0"], out["gx"], out["gm"] = m.quality(grad=True)
        m.smooth(kind=LAPLACE)
        m.smooth(kind=GRADIENT)
        m.sweep(0)
    out["Q"], out["qmin"] = m.quality()
    out.update(_export(m, state["buffers"]))
    m.close()
    return out


# ---- what a pass cannot do without ----------------------------------------------

def work(case):
    """Bytes: each input array read once and each output array written once.
    Flops: about 60 for an element's quality, 250 with its gradient, 100 for a
    vertex's move, 300 for a vertex that is offered a collapse or a flip."""
    kind = case["kind"]
    if kind in ("tet", "tetpsi"):
        V, T = case["n"] ** 3, 6 * (case["n"] - 1) ** 3
        out = case["target"] if kind == "tetpsi" else case["ratio"] * T
        return dict(bytes=V * 73 + T * 16 + out * (16 + 73 / 5.0), flops=(V + out / 5) * 1000)
    if kind == "batch":  # n log-uniform: the mean of n^2
        lo, hi = case["nmin"], case["nmax"]
        V = case["count"] * (hi * hi - lo * lo) / (2.0 * math.log(hi / lo))
        return dict(bytes=V * 65 * 1.6, flops=V * 400 * case["sweeps"])
    V, T = case["n"] ** 2, 2 * (case["n"] - 1) ** 2
    whole = V * 41 + T * 12
    if kind == "quality":
        return dict(bytes=whole + V * 40, flops=T * 250)
    if kind == "smooth":
        return dict(bytes=whole + V * 16, flops=V * 700 * case["sweeps"])
    if kind == "psi":
        return dict(bytes=2.0 * case["target"] * 32.5, flops=case["target"] * 700)
    if kind == "step":
        return dict(bytes=whole + V * 40, flops=T * 310 + V * 1700)
    return dict(bytes=whole * (1.0 + case.get("ratio", 0.0)), flops=V * 400)


# ---- in 64 bits, without the library --------------------------------------------

def _quality64(xy, tri, met, kind):
    """Sum and minimum of the element quality, plain torch."""
    p, m = [xy[tri[:, k]] for k in range(3)], (met[tri[:, 0]] + met[tri[:, 1]] + met[tri[:, 2]]) / 3.0
    a, b, c = m[:, 0], m[:, 1], m[:, 2]

    def len2(u, v):
        d = v - u
        return a * d[:, 0] ** 2 + 2.0 * b * d[:, 0] * d[:, 1] + c * d[:, 1] ** 2

    e1, e2 = p[1] - p[0], p[2] - p[0]
    area = 0.5 * (e1[:, 0] * e2[:, 1] - e2[:, 0] * e1[:, 1])
    root = torch.sqrt(a * c - b * b)
    L = [len2(p[0], p[1]), len2(p[1], p[2]), len2(p[2], p[0])]
    if kind == MEAN:
        q = 4.0 * math.sqrt(3.0) * root * area / (L[0] + L[1] + L[2])
    else:
        P = L[0].sqrt() + L[1].sqrt() + L[2].sqrt()
        x = P / 3.0
        f = torch.minimum(x, 1.0 / x)
        q = 12.0 * math.sqrt(3.0) * root * area / (P * P) * (f * (2.0 - f)) ** 3
    return q.sum(), q.min()


def exact(case, seed):
    """The functional and its gradient of the inputs; adapted meshes are
    products of the method's own decisions and have no closed form."""
    if case["kind"] not in ("quality", "step"):
        return None
    mi = _grid(case, seed)
    xy, met = _dev(mi.xy).requires_grad_(), _dev(mi.metric).requires_grad_()
    Q, qmin = _quality64(xy, _dev(mi.tri).long(), met, case.get("quality", MEAN))
    gx, gm = torch.autograd.grad(Q, (xy, met))
    if case["kind"] == "quality":
        return dict(Q=Q.detach(), gx=gx, gm=gm)
    none = dict.fromkeys(("Q", "qmin", "V", "T", "xy", "elements", "metric", "tags"))
    return dict(none, Q0=float(Q), qmin0=float(qmin), gx=gx, gm=gm)
