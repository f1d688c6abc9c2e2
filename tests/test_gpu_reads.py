"""Packed reads and loads at the sizes where they change route: a state just
below and just above what the page-locked block takes (for the fluid state
26,188 particles, for a checkpoint about 26,150 slots), and a read in the
middle of a ring. The fluid state is compared with the checkpoint's own
arrays, decoded here, bit for bit."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

wc = pytest.importorskip("paper_2609_05494_amd")


def _decode(s, blob):
    cfg, N, ng = s.cfgs[0], s.n_slots, s.ng
    o = len(blob) - (N * (4 + 4 + 16 + 16 + 2) + ng * 4)
    cell = np.frombuffer(blob, np.uint32, N, o)
    pid = np.frombuffer(blob, np.uint32, N, o + 4 * N)
    pv = np.frombuffer(blob, np.float32, 4 * N, o + 8 * N).reshape(N, 4).astype(np.float64)
    rho = np.frombuffer(blob, np.float32, 4 * N, o + 24 * N).reshape(N, 4)[:, 0].astype(np.float64)
    g, dc = cfg["ghost_layers"] * cfg["dx"], cfg["cell_size"]
    ncx = int(np.ceil((cfg["L"] + 2 * g) / dc))
    x, y = -g + (cell % ncx) * dc + pv[:, 0], -g + (cell // ncx) * dc + pv[:, 1]
    f = pid < s.nf
    out = np.empty((5, s.nf))
    out[:, pid[f]] = np.stack([x, y, pv[:, 2], pv[:, 3], rho])[:, f]
    return out


@pytest.mark.parametrize("nx,ny", [(170, 140), (175, 141), (187, 140), (187, 141)])
def test_reads_and_loads_around_the_block_size(nx, ny):
    cfg = workloads.base(nx * 1e-3, ny * 1e-3, 1e-3, 4e-3, 600.0)
    cfg = dict(cfg, disk_R=0.0, n_disk_ghosts=0, init_mode=1)
    print(f"[gpu] {nx}x{ny}", flush=True)
    s = wc.Solver(cfg, "cuda:0")
    s.step(7)
    blob = s.save_state()
    assert np.array_equal(np.stack(s.fluid()[1]), _decode(s, blob))
    s.step(13)
    a, p = s.fluid(), s.read_probes()
    s.load_state(blob)
    assert np.array_equal(np.stack(s.fluid()[1]), _decode(s, blob))
    s.step(13)
    b, q = s.fluid(), s.read_probes()
    assert a[0] == b[0] and all(np.array_equal(u, v) for u, v in zip(a[1], b[1]))
    # the rows after the load are the run's last ones
    assert all(np.array_equal(u[7:], v) for u, v in zip(p, q))
    s.close()
