"""The pair pass's scan where its groups, passes and hit lists end: particles
scattered without a lattice, sparse rows (groups cut by their width), cells
of many particles (several passes, a pass with more hits than a list takes).
Rates against the FP64 oracle on the same state, in-support neighbour sets
against its O(N^2) search."""
import numpy as np
import pytest

import oracle
import workloads
from tests import shared_state

pytestmark = pytest.mark.gpu

wc = pytest.importorskip("paper_2609_05494_amd")

# the bar of every one-evaluation rate test: 1e-4 of the field's maximum
RATE_BAR = 1e-4


def _cfg(kernel_type):
    return dict(workloads.tiny(L=0.052, W=0.026, R=0.003), kernel_type=kernel_type)


def _positions(kind, cfg, n, rng):
    L, W, dc = cfg["L"], cfg["W"], cfg["cell_size"]
    x, y = rng.uniform(0.1e-3, L - 0.1e-3, n), rng.uniform(0.1e-3, W - 0.1e-3, n)
    lo = -cfg["ghost_layers"] * cfg["dx"]

    def crowd(ids, cx, cy, per_cell):
        # per_cell particles in each of the cells from (cx, cy) on, left to right
        k = np.arange(ids.size) // per_cell
        x[ids] = lo + (cx + k % 3 + rng.uniform(0.02, 0.98, ids.size)) * dc
        y[ids] = lo + (cy + k // 3 + rng.uniform(0.02, 0.98, ids.size)) * dc

    if kind == "sparse":
        # one particle in eight stays scattered; the others stand in a band of
        # cells, so that most cells outside it are empty
        band = np.arange(n) % 8 != 0
        x[band] = rng.uniform(0.75 * L, L - 0.1e-3, band.sum())
    elif kind == "crowded":
        # 3 x 3 cells of 50: a middle particle has some 200 neighbours
        crowd(np.arange(450), 8, 3, 50)
    return x, y


@pytest.mark.parametrize("kernel_type", [0, 1])
@pytest.mark.parametrize("kind", ["scattered", "sparse", "crowded"])
def test_scan_of_irregular_states(kind, kernel_type):
    cfg = _cfg(kernel_type)
    print(f"[gpu] {kind}, kernel {kernel_type}", flush=True)
    s, o = wc.Solver(cfg, "cuda:0"), oracle.Oracle(cfg)
    rng = np.random.default_rng(7)
    n = s.nf
    x, y = _positions(kind, cfg, n, rng)
    v = rng.normal(0.0, 30.0, (2, n))
    rho = 1000.0 * (1.0 + rng.normal(0.0, 0.01, n))
    st = shared_state.round_state(cfg, x, y, v[0], v[1], rho)
    s.set_fluid(0.0, *st)
    o.set_fluid(0.0, *st)
    g, w = s.export_rates(), o.eval_rates()
    for a, b in (("ax", "ay"), ("Vx", "Vy")):
        d = np.hypot(g[a] - w[a], g[b] - w[b]).max()
        assert d <= RATE_BAR * np.hypot(w[a], w[b]).max(), (a, d)
    assert np.abs(g["drho"] - w["drho"]).max() <= RATE_BAR * np.abs(w["drho"]).max()
    o.eval_rates()
    gx, gy, _ = o.ghosts()
    px, py = np.concatenate([st[0], gx]), np.concatenate([st[1], gy])
    h2 = 4.0 * (cfg["h_over_dx"] * cfg["dx"]) ** 2
    d2 = (px[:n, None] - px[None]) ** 2 + (py[:n, None] - py[None]) ** 2
    inside, near = d2 < h2, np.abs(d2 - h2) < 1e-5 * h2
    inside[np.arange(n), np.arange(n)] = False
    if (inside | near).sum(axis=1).max() <= 64:  # (a list holds 64 ids)
        for k, got in enumerate(s.export_neighbour_lists()):
            hit = np.zeros(px.size, bool)
            hit[got] = True
            assert got.size == hit.sum() and not ((hit != inside[k]) & ~near[k]).any(), k
    else:
        assert kind != "scattered"
    s.close()
