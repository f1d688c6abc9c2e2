"""Which neighbours the pair pass sums where a wave's passes end: cells of up to
60 particles, a slot with more hits in a pass than its list takes (the pass is
then halved), and sparse rows. Every particle's neighbour count against the
O(N^2) search (the export counts past the 64 ids that it records), and the
ids of the particles that have no more than 64; pairs within 1e-5 of the
support's edge may go either way in FP32."""
import ctypes as C

import numpy as np
import pytest

import oracle
from tests import shared_state
from tests.test_gpu_pair_scan import _cfg, _positions

pytestmark = pytest.mark.gpu

wc = pytest.importorskip("paper_2609_05494_amd")


def _state(kind, cfg, n, rng):
    x, y = _positions("sparse" if kind == "sparse" else "crowded", cfg, n, rng)
    if kind == "packed":
        # 5 x 2 cells of 58: five passes of 128 entries
        dc, lo = cfg["cell_size"], -cfg["ghost_layers"] * cfg["dx"]
        x, y = rng.uniform(0.030, 0.051, n), rng.uniform(0.1e-3, cfg["W"] - 0.1e-3, n)
        k = np.arange(580) // 58
        x[:580] = lo + (4 + k % 5 + rng.uniform(0.02, 0.98, 580)) * dc
        y[:580] = lo + (4 + k // 5 + rng.uniform(0.02, 0.98, 580)) * dc
    return x, y


@pytest.mark.parametrize("kernel_type", [0, 1])
@pytest.mark.parametrize("kind", ["sparse", "crowded", "packed"])
def test_neighbours_of_crowded_cells(kind, kernel_type):
    cfg = _cfg(kernel_type)
    print(f"[gpu] neighbours, {kind}, kernel {kernel_type}", flush=True)
    s, o = wc.Solver(cfg, "cuda:0"), oracle.Oracle(cfg)
    rng = np.random.default_rng(7)
    n = s.nf
    x, y = _state(kind, cfg, n, rng)
    st = shared_state.round_state(cfg, x, y, *rng.normal(0.0, 30.0, (2, n)), np.full(n, 1000.0))
    s.set_fluid(0.0, *st)
    o.set_fluid(0.0, *st)
    o.eval_rates()
    gx, gy, _ = o.ghosts()
    px, py = np.concatenate([st[0], gx]), np.concatenate([st[1], gy])
    h2 = 4.0 * (cfg["h_over_dx"] * cfg["dx"]) ** 2
    d2 = (px[:n, None] - px[None]) ** 2 + (py[:n, None] - py[None]) ** 2
    d2[np.arange(n), np.arange(n)] = np.inf
    sure, maybe = d2 < (1 - 1e-5) * h2, d2 < (1 + 1e-5) * h2
    assert maybe.sum(axis=1).max() > 64
    count, ids = np.zeros(n, np.int32), np.zeros((n, 64), np.uint32)
    r = wc.lib().wcsph_export_neighbour_lists(s.handle, count.ctypes.data_as(C.POINTER(C.c_int)),
                                              ids.ctypes.data_as(C.POINTER(C.c_uint)), 64, n)
    assert r == wc.E_RANGE  # (some have more than 64)
    assert np.all(sure.sum(axis=1) <= count) and np.all(count <= maybe.sum(axis=1))
    for k in np.flatnonzero(count <= 64):
        got = ids[k, :count[k]]
        assert np.unique(got).size == got.size and maybe[k][got].all() and not np.setdiff1d(np.flatnonzero(sure[k]), got).size, k
    s.close()
