"""Flat chunked tiles whose rows have no connections, the last tile of the last
network among them, against the fp64 oracle within the per-row bound of
test_gpu_parity.py."""
import numpy as np
import pytest

from paper_1612_01501_amd import inputs as I
from test_gpu_gap_forms import check_gap, infoli  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("weights", [False, True])
@pytest.mark.parametrize("n,linked,rows", [(300, 44, 8), (600, 256, 64), (600, 300, 256), (9000, 8, 256)])
def test_isolated_last_rows(infoli, o64, n, linked, rows, weights):
    """`linked` cells of 16 connections each (two whole chunks) ahead of rows
    without any."""
    shift = np.array([-8, -7, -6, -5, -4, -3, -2, -1, 1, 2, 3, 4, 5, 6, 7, 8])
    deg = 16 if linked >= 17 else 4
    cols = [np.unique((i + (shift if deg == 16 else np.array([1, 2, 3, 4]))) % linked) for i in range(linked)]
    rp = np.zeros(n + 1, np.int64)
    rp[1:linked + 1] = np.cumsum([len(c) for c in cols])
    rp[linked + 1:] = rp[linked]
    col = np.concatenate(cols).astype(np.int32)
    rs = I.rng(n)
    net = I.Network(n=n, conn="csr", g=0.04, row_ptr=rp, col=col, jitter=rs.uniform(-15, 15, (3, n)),
                    w_csr=rs.uniform(0.02, 0.06, len(col)).astype(np.float32) if weights else None)
    x0 = infoli.initial_state(net)
    first = I.Network(n=33, conn="none")
    for nets in ([net], [first, net]):
        sim = infoli.Simulator(nets, init_states=[infoli.initial_state(first)] * (len(nets) - 1) + [x0], csr_path=4,
                               tile_rows=rows, step_mode="graph")
        assert sim.gap_path(len(nets) - 1) == ("csr_chunked", False)
        check_gap(sim, len(nets) - 1, net, x0[0], o64)
        sim.step(2)
        sim.sync()
        sim.close()


def test_chunked_rows_past_the_flat_tiles(infoli, o64, tmp_path, monkeypatch):
    """Tiles of 256 rows whose chunk sums do not fit LDS beside the voltages:
    the lane groups gather from memory, with no copy of the voltages that
    nothing reads (the tuner times none such)."""
    n, deg = 8192, 1000
    rp, col = I.erdos_renyi_csr(n, deg / (n - 1), 3)
    net = I.Network(n=n, conn="csr", g=0.04 * 96 / deg, row_ptr=rp, col=col, jitter=I.voltage_jitter(n, 5, 15.0))
    x0 = infoli.initial_state(net)
    sim = infoli.Simulator(net, init_states=[x0], csr_path=4, tile_rows=256, step_mode="graph")
    assert sim.gap_path(0) == ("csr_chunked", False)
    check_gap(sim, 0, net, x0[0], o64)
    sim.close()
    log = tmp_path / "log.txt"
    monkeypatch.setenv("INFOLI_TUNE_LOG", str(log))
    sim = infoli.Simulator(net, init_states=[x0], step_mode="graph", autotune=2)
    check_gap(sim, 0, net, x0[0], o64)
    sim.close()
    shapes = [ln.split(" shape ")[1].split(":")[0].split() for ln in log.read_text().splitlines() if " shape " in ln]
    rows = [s for s in shapes if s[3] == "path3"]
    assert any(s[1] == "R256" and s[0] != "L64" for s in rows)      # lane groups, timed
    assert all(s[2] == "lds0" or s[0] == "L64" for s in rows)       # staged by the flat tiles alone
