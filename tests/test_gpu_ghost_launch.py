"""Ghosts in the sort's launch against ghosts in a launch of their own, over
every form and option that both serve: states, histories, every diagnostic
(the audit's sums, the ring's work), impulse and gradient are the same bit for
bit, also when the launch changes in the middle of a run."""
import time

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

wc = pytest.importorskip("paper_2609_05494_amd")

FORMS = {
    "plain": lambda c: c,
    "no_disk": lambda c: dict(c, disk_R=0.0, n_disk_ghosts=0, init_mode=1),
    "audit": lambda c: dict(c, audit=1),
    "audit_cubic_beta": lambda c: dict(c, audit=1, kernel_type=1, beta=1.0),
    "beta": lambda c: dict(c, beta=1.0),
    "cubic": lambda c: dict(c, kernel_type=1),
    "mg": workloads.mie_grueneisen,
    "mg_inverse_cubic": lambda c: dict(workloads.mie_grueneisen(c), kernel_type=1, ghost_rho_mode=1),
    "two_way": workloads.two_way,
    "two_way_audit": lambda c: dict(workloads.two_way(c), audit=1),
    "drag": lambda c: dict(c, kin_mode=1, kin_coef=3.0),
    "axisym": workloads.axisymmetric,
    "wide": lambda c: dict(c, h_over_dx=2.0, cell_size=workloads._cell_size(c["dx"], 2.0), ghost_layers=4),
    "dense_cells": lambda c: dict(c, cell_size=float(np.float32(5.5 * c["dx"])), n_disk_ghosts=40),
    "crowded_ring": lambda c: dict(c, n_disk_ghosts=256),
    "axisym_two_way": lambda c: workloads.axisymmetric(dict(c, kin_mode=2)),
}


def _same(a, b):
    for u, v in zip(a.read_probes() + a.disk_state(), b.read_probes() + b.disk_state()):
        assert np.array_equal(u, v)
    da, db = a.read_diagnostics(), b.read_diagnostics()
    for k in da:
        assert np.array_equal(da[k], db[k]), k
    (ta, fa), (tb, fb) = a.fluid(), b.fluid()
    assert ta == tb
    for u, v in zip(fa, fb):
        assert np.array_equal(u, v)


def _pair(cfg):
    a, b = wc.Solver(cfg, "cuda:0"), wc.Solver(cfg, "cuda:0")
    a.set_ghost_launch(False)
    b.set_ghost_launch(True)
    assert not a.set_ghost_launch(False) and b.set_ghost_launch(True)
    return a, b


@pytest.mark.parametrize("form", FORMS)
def test_both_launches_give_the_same_run(form):
    cfg = FORMS[form](workloads.C1())
    print(f"[gpu] both ghost launches, {form}", flush=True)
    a, b = _pair(cfg)
    for s in (a, b):
        s.step(67)  # past the 5 us ramp: a two-way disk is coupled by then
    _same(a, b)
    # the other way round from here, and back
    for s, first in ((a, True), (b, False)):
        s.set_ghost_launch(first)
        s.step(14)
        s.set_ghost_launch(not first)
        s.step(9)
    _same(a, b)
    a.close()
    b.close()


def test_both_launches_follow_a_table_and_fixed_steps():
    cfg = dict(workloads.C1(), kin_mode=3)
    print("[gpu] both ghost launches, tabulated motion", flush=True)
    a, b = _pair(cfg)
    for s in (a, b):
        s.set_kinematics_table([(0.0, 4e-3, 0.0, 4e7), (4e-6, 4.3e-3, 160.0, 1e7), (8e-6, 5.1e-3, 200.0, -1e6)])
        s.step(30)
        s.set_dt_table(np.full(40, 1.1e-7))
        s.step(45)
        s.set_coefficients(0.2, 0.05, 1500.0)
        s.step(6)
    _same(a, b)
    a.close()
    b.close()


@pytest.mark.parametrize("ckpt", [7, 25])
def test_both_launches_tape_the_same_run(ckpt):
    cfg = workloads.C1()
    print(f"[gpu] both ghost launches, adjoint, checkpoint every {ckpt}", flush=True)
    a, b = _pair(cfg)
    out = []
    for s in (a, b):
        s.step(60)
        blob = s.save_state()
        s.set_dt_table(np.full(25, 1.1e-7))
        s.load_state(blob)
        J = s.adj_forward(25, ckpt)
        out.append(np.append(s.adj_backward(1.0), J))
    assert np.all(np.isfinite(out[0])) and np.any(out[0][:3] != 0.0)
    assert np.array_equal(*out)
    _same(a, b)
    a.close()
    b.close()


def test_contexts_with_one_ghost_launch_refuse_the_choice():
    for cfg in ([workloads.tiny()], workloads.paper_scheme(workloads.tiny())):
        s = wc.Solver(cfg, "cuda:0")
        with pytest.raises(wc.WcsphError) as e:
            s.set_ghost_launch(True)
        assert e.value.status == wc.E_INVALID
        s.step(2)
        s.close()


# 763, 772, 759 and 770 blocks: either side of three per compute unit (768)
@pytest.mark.parametrize("nx,h_over_dx,own", [(428, 1.0, False), (432, 1.0, True), (532, 1.3, False), (536, 1.3, True)])
def test_choice_on_either_side_of_the_line(nx, h_over_dx, own):
    cfg = workloads.base(nx * 1e-3, nx // 2 * 1e-3, 1e-3, 6e-3, 900.0)
    cfg = dict(cfg, h_over_dx=h_over_dx, cell_size=workloads._cell_size(1e-3, h_over_dx))
    print(f"[gpu] {nx}x{nx // 2}, h/dx {h_over_dx}", flush=True)
    a, b, c = wc.Solver(cfg, "cuda:0"), wc.Solver(cfg, "cuda:0"), wc.Solver([cfg], "cuda:0")
    assert b.set_ghost_launch(not own) == own
    for s in (a, b, c):
        s.step(23)
    _same(c, a)
    c.close()
    d = wc.Solver(cfg, "cuda:0")
    d.step(23)
    _same(d, b)
    for s in (a, b, d):
        s.close()


def _channel(nx, ny, dx, h_over_dx=1.3, **kw):
    cfg = workloads.base(nx * dx, ny * dx, dx, 12 * dx, 900.0)
    return dict(cfg, h_over_dx=h_over_dx, **dict(dict(cell_size=workloads._cell_size(dx, h_over_dx)), **kw))


CROWDS = {
    # probes of both walls: 852 particles in one block, 88 -> 116 us a step
    "narrow": _channel(1263, 63, 0.5e-3, 2.0, ghost_layers=4),
    # left and right wall with the ring between them: 344, 60 -> 71 us
    "ring": dict(workloads.tiny(), n_disk_ghosts=150),
    # 30 particles a cell around a run of ring ghosts: 382, 92 -> 164 us
    "dense": _channel(346, 173, 0.5e-3, cell_size=float(np.float32(2.75e-3))),
}


@pytest.mark.parametrize("crowd", CROWDS)
def test_no_block_holds_up_the_launch(crowd):
    """A block of the sort's launch takes items whose surroundings it can stage
    at once (320 particles). The figures above are a launch of their own ->
    the sort's with such a block; without, the sort's launch is the faster."""
    print(f"[gpu] {crowd}", flush=True)
    s = wc.Solver(CROWDS[crowd], "cuda:0")
    s.step(100)
    best = {}
    for own in (True, False) * 4:
        s.set_ghost_launch(own)
        s.step(20)
        s.synchronize()
        t0 = time.perf_counter()
        s.step(100)
        s.synchronize()
        best[own] = min(best.get(own, np.inf), time.perf_counter() - t0)
    s.close()
    print(f"us a step: own launch {1e4 * best[True]:.1f}, in the sort's {1e4 * best[False]:.1f}")
    assert best[False] < 1.12 * best[True]
