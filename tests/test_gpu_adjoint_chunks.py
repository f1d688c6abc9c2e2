"""The reverse sweep's fluid pass over more than two candidate chunks (128
candidates per slot and chunk): cells wider than the support hold about 225
and 310 candidates around a particle. Gradient against the oracle's FP64
tangent, with the bar of the small adjoint case."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

wc = pytest.importorskip("paper_2609_05494_amd")


@pytest.mark.parametrize("h_over_dx,edge", [(1.3, 5.0), (2.0, 5.9)])
def test_adjoint_of_wide_cells(h_over_dx, edge):
    base = workloads.tiny(L=0.030, W=0.021, v0=600.0)
    # (40 ring ghosts: a hundred would crowd one cell beyond its 64 places)
    cfg = dict(base, h_over_dx=h_over_dx, cell_size=float(np.float32(edge * base["dx"])), n_disk_ghosts=40,
               ghost_layers=int(np.ceil(2 * h_over_dx)))
    n = 20
    o = oracle.Oracle(cfg)
    o.step(n)
    dt = o.probes()[1]
    print(f"[gpu] adjoint, h/dx {h_over_dx}, cells of {edge} dx", flush=True)
    s = wc.Solver(cfg, "cuda:0")
    c = s.export_cells()["cell_start"]
    ncx = int(np.ceil((cfg["L"] + 2 * cfg["ghost_layers"] * cfg["dx"]) / cfg["cell_size"]))
    per = np.diff(c).reshape(-1, ncx)
    around = sum(per[1 + i:per.shape[0] - 1 + i, 1 + j:ncx - 1 + j] for i in (-1, 0, 1) for j in (-1, 0, 1))
    assert around.max() > (256 if h_over_dx == 2.0 else 128)
    s.set_dt_table(dt)
    s.adj_forward(n, n)
    g = s.adj_backward(1.0)
    s.close()
    _, go = oracle.tangent_J(cfg, dt)
    print(f"grad {g} oracle {go}; rel {np.abs(g - go) / np.abs(go)}")
    assert np.all(np.abs(g - go) <= 2e-3 * np.abs(go))
