"""A state set from the host after a run replaces everything the run left: the
steps that follow are those of a new context, bit for bit, whatever the step
count was (the leapfrog alternates two bucket sets from step to step)."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

wc = pytest.importorskip("paper_2609_05494_amd")


@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("before", [1, 2, 3])
def test_set_fluid_after_a_run(before, scheme):
    cfg = workloads.C1()
    if scheme == 1:
        cfg = workloads.paper_scheme(cfg)
    print(f"[gpu] scheme {scheme}, {before} steps before set_fluid", flush=True)
    a, b = wc.Solver(cfg, "cuda:0"), wc.Solver(cfg, "cuda:0")
    a.step(20)
    t, f = a.fluid()
    a.close()
    c = wc.Solver(cfg, "cuda:0")
    b.step(before)
    for s in (b, c):
        s.set_fluid(t, *f)
        s.step(5)
    assert b.fluid()[0] == c.fluid()[0]
    for u, v in zip(b.fluid()[1] + [b.internal_energy()], c.fluid()[1] + [c.internal_energy()]):
        assert np.array_equal(u, v)
    for u, v in zip(b.read_probes(), c.read_probes()):
        assert np.array_equal(u, v)
    b.close()
    c.close()
