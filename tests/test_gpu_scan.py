"""Ordered scans at the edges of their splits (one work-group, several, coarser
sums, sums scanned by themselves): a selection through a colouring, and the row
headers, counts and places of a refinement pass, on grids with known answers."""
import numpy as np
import pytest
import torch

from paper_1505_04694_amd import pmesh

pytestmark = pytest.mark.gpu


def grid(n):
    """n x n vertices, two triangles a square, on the device."""
    g = torch.arange(n, device="cuda", dtype=torch.float64) / (n - 1)
    xy = torch.stack([g.repeat(n), g.repeat_interleave(n)], 1)
    i = torch.arange((n - 1) * (n - 1), device="cuda", dtype=torch.int32)
    a = (i // (n - 1)) * n + i % (n - 1)
    tri = torch.stack([torch.stack([a, a + 1, a + n + 1], 1), torch.stack([a, a + n + 1, a + n], 1)], 1).reshape(-1, 3)
    return xy.contiguous(), tri.contiguous()


def star_edges(n, p):
    """The edges at vertex p, smaller id first."""
    x, y = p % n, p // n
    out = []
    for dx, dy in ((1, 0), (0, 1), (1, 1), (-1, 0), (0, -1), (-1, -1)):
        if 0 <= x + dx < n and 0 <= y + dy < n:
            q = (y + dy) * n + x + dx
            out.append((min(p, q), max(p, q)))
    return out


def star_elements(n, p):
    x, y = p % n, p // n
    at = [(dx, dy) for dx, dy in ((0, 0), (-1, 0), (0, -1), (-1, -1)) if 0 <= x + dx < n - 1 and 0 <= y + dy < n - 1]
    # both triangles of a square hold its first and last corner, one each the others
    return sum(2 if d in ((0, 0), (-1, -1)) else 1 for d in at)


@pytest.mark.parametrize("n", [2, 16, 17, 46, 91, 1448, 1449, 2897])
def test_selection_and_refinement_places(n):
    V = n * n
    xy, tri = grid(n)
    metric = torch.tensor([1.0, 0.0, 1.0], device="cuda", dtype=torch.float64).repeat(V, 1)
    # far apart, the first and the last slots and one at each split among them
    picks = {0, V - 1}
    for k in (255, 256, 2047, 2048, V // 3, V // 2, 1024 * 8192):
        p = min(k, V - 1)
        if all(max(abs(p % n - q % n), abs(p // n - q // n)) > 2 for q in picks):
            picks.add(p)
    picks = sorted(picks)
    metric[torch.tensor(picks, device="cuda")] = torch.tensor([100.0, 0.0, 100.0], device="cuda", dtype=torch.float64)
    m = pmesh.Mesh(xy, tri, metric, seed=3)
    active = np.zeros(V, np.uint8)
    active[picks] = 1
    colours, _ = m.colour(active)
    assert np.array_equal(np.flatnonzero(np.asarray(colours) >= 0), picks)
    h2 = 1.0 / (n - 1) ** 2
    m.refine(L_up2=10.0 * h2, max_passes=1)
    edges = sorted({e for p in picks for e in star_edges(n, p)})
    assert m.sizes() == (V + len(edges), len(tri) + 2 * sum(star_elements(n, p) for p in picks) - (n == 2) * 2)
    e = m.export()
    x = xy.cpu().numpy()
    mid = np.array([(x[a] + x[b]) * 0.5 for a, b in edges])
    assert np.array_equal(np.asarray(e["xy"])[V:], mid)
    m.close()
