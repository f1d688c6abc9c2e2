"""The reverse sweep's fluid pass where its candidate chunks (128 per slot)
end: supports of fewer, just over and well over one chunk of candidates.
Gradient against the oracle's FP64 tangent, with the bar of the small
adjoint case. (The impulse itself is the forward run's: at h/dx 1.1 the
pressure has hardly reached the probes, and FP32 rounding of the state alone
moves the oracle's J by 6.5e-3.)"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

wc = pytest.importorskip("paper_2609_05494_amd")


@pytest.mark.parametrize("h_over_dx", [1.1, 1.9, 2.0])
def test_adjoint_of_wide_supports(h_over_dx):
    base = workloads.tiny(L=0.030, W=0.021, v0=600.0)
    cfg = dict(base, h_over_dx=h_over_dx, cell_size=workloads._cell_size(base["dx"], h_over_dx),
               ghost_layers=int(np.ceil(2 * h_over_dx)))
    n = 20
    o = oracle.Oracle(cfg)
    o.step(n)
    dt = o.probes()[1]
    print(f"[gpu] adjoint, h/dx {h_over_dx}", flush=True)
    s = wc.Solver(cfg, "cuda:0")
    s.set_dt_table(dt)
    s.adj_forward(n, n)
    g = s.adj_backward(1.0)
    s.close()
    _, go = oracle.tangent_J(cfg, dt)
    print(f"grad {g} oracle {go}; rel {np.abs(g - go) / np.abs(go)}")
    assert np.all(np.abs(g - go) <= 2e-3 * np.abs(go))
