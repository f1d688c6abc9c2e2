"""Checkpoints of more than the page-locked block takes (1 MiB: copied array by
array) with each array that only some contexts have: a batch's instance tags,
the audit's sums, the leapfrog's internal energy. The steps after a load are
those of the run that saved, bit for bit, in the same and in a new context;
long reads of an instance of a batch and of the internal energy equal the
checkpoint's own arrays."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

wc = pytest.importorskip("paper_2609_05494_amd")


HEAD, CLOCK = 64, 184  # bytes of a checkpoint's header and of one clock


def _channel(nx, ny, **kw):
    return workloads.base(nx * 1e-3, ny * 1e-3, 1e-3, 5e-3, 900.0, **kw)


FORMS = {
    "batch": [_channel(160, 90), _channel(171, 83, alpha=0.3)],
    "audit": dict(_channel(190, 151), audit=1),
    "leapfrog": workloads.paper_scheme(_channel(190, 151)),
    "leapfrog_batch": [workloads.paper_scheme(_channel(160, 90)), workloads.paper_scheme(_channel(171, 83))],
}


def _everything(s):
    out = []
    for i in range(s.n_inst):
        t, f = s.fluid(i)
        out += [t, *f, s.internal_energy(i)]
    for i in range(s.n_inst):
        d = s.read_diagnostics(i)
        out += [d[k] for k in sorted(d)] + list(s.read_probes(i))
    return out


@pytest.mark.parametrize("form", FORMS)
def test_a_long_checkpoint_restores_every_array(form):
    cfg = FORMS[form]
    print(f"[gpu] long checkpoint, {form}", flush=True)
    a = wc.Solver(cfg, "cuda:0")
    a.step(23)
    blob = a.save_state()
    assert len(blob) > 1 << 20
    for i in range(a.n_inst):
        a.read_probes(i), a.read_diagnostics(i)
    a.step(17)
    ref = _everything(a)
    b = wc.Solver(cfg, "cuda:0")
    b.step(3)
    for s in (a, b):
        s.load_state(blob)
        # (the arrays after the header and the clocks: a load recomputes the clock's v_max)
        assert s.save_state()[HEAD + s.n_inst * CLOCK:] == blob[HEAD + s.n_inst * CLOCK:]
        s.step(17)
        got = _everything(s)
        assert len(got) == len(ref) and all(np.array_equal(u, v) for u, v in zip(got, ref))
        s.close()


def test_long_reads_of_one_instance():
    cfgs = [workloads.tiny(), _channel(190, 151), _channel(80, 40)]
    print("[gpu] long read, batch", flush=True)
    b = wc.Solver(cfgs, "cuda:0")
    b.step(12)
    for i, cfg in enumerate(cfgs):
        s = wc.Solver(cfg, "cuda:0")
        s.step(12)
        assert s.fluid()[0] == b.fluid(i)[0]
        assert all(np.array_equal(u, v) for u, v in zip(s.fluid()[1], b.fluid(i)[1]))
        s.close()
    b.close()


def test_long_read_of_the_internal_energy():
    print("[gpu] long read, internal energy", flush=True)
    s = wc.Solver(workloads.paper_scheme(_channel(520, 260)), "cuda:0")
    assert s.nf * 8 > 1 << 20
    s.step(15)
    e = s.internal_energy()
    blob, N = s.save_state(), s.n_slots
    o = len(blob) - (N * (4 + 4 + 16 + 16 + 2 + 4) + s.ng * 4)
    pid = np.frombuffer(blob, np.uint32, N, o + 4 * N)
    want = np.full(s.nf, np.nan)
    f = pid < s.nf
    want[pid[f]] = np.frombuffer(blob, np.float32, N, len(blob) - 4 * N)[f]
    assert np.any(e > 0.0) and np.array_equal(e, want)
    s.close()
