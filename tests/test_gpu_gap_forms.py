"""Gap currents of the coupling forms at the sizes where their tiles, column
stretches and voltage ranges begin and end, against the fp64 oracle within
the per-row bound of test_gpu_parity.py (1e-5 of the row's sum of |terms|
plus eight ulp of max|Vd| times the row's weight sum)."""
import numpy as np
import pytest

from paper_1612_01501_amd import inputs as I
from test_gpu_parity import gap_bound

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def infoli():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1612_01501_amd import infoli as mod
    mod.lib()
    return mod


def check_gap(sim, k, net, vd, o64):
    got = sim.read_gap_current(k).astype(np.float64)
    ref = o64.gap(net, vd.astype(np.float64))
    tol = gap_bound(net, vd)
    err = np.abs(got - ref) / tol
    assert np.all(err <= 1.0), (net.label or net.conn, net.n, int(np.argmax(err)), float(err.max()))


@pytest.mark.parametrize("gap", ["rgj", "sgj"])
@pytest.mark.parametrize("n,rows", [(3, 0), (255, 0), (256, 7), (257, 0), (511, 5), (1024, 0), (1027, 16)])
def test_dense_stretches(infoli, o64, n, rows, gap):
    """Column stretches of 256 in four-row passes: partial stretches, row
    counts that are no multiple of four, and a second network whose weights
    and cells start at odd offsets."""
    rs = I.rng(n + 7)
    nets = [I.Network(n=m, conn="dense", w_dense=rs.uniform(0, 0.05, (m, m)).astype(np.float32), gap=gap,
                      jitter=rs.uniform(-15, 15, (3, m))) for m in (n, 65)]
    x0s = [infoli.initial_state(net) for net in nets]
    sim = infoli.Simulator(nets[::-1], init_states=x0s[::-1], tile_rows=rows, step_mode="graph")
    for k, (net, x0) in enumerate(zip(nets[::-1], x0s[::-1])):
        check_gap(sim, k, net, x0[0], o64)
    sim.close()


# name, sizes, voltages: one tile and several, the edge of a share, one and many
# groups of grid points, voltages at whole millivolts, tiles too wide for the grid
SPREADS = {
    "jitter": lambda rs, n: -60.0 + rs.uniform(-1.0, 1.0, n),
    "wide": lambda rs, n: rs.uniform(-95.0, 60.0, n),
    "near": lambda rs, n: -60.0 + rs.uniform(-1e-4, 1e-4, n),
    "whole": lambda rs, n: rs.integers(-70, -40, n).astype(np.float64),
    "far": lambda rs, n: np.where(rs.random(n) < 0.02, rs.uniform(-4000.0, 4000.0, n), rs.uniform(-61.0, -59.0, n)),
}


@pytest.mark.parametrize("spread", sorted(SPREADS))
@pytest.mark.parametrize("n", [512, 513, 1000, 4095, 4096, 8193, 16385])
def test_voltage_grid(infoli, o64, n, spread):
    """All-to-all networks on the voltage grid, alone (each tile its own sums
    below 4,096 cells, the sums ahead of the step from there on) and in a
    batch behind an odd number of cells."""
    rs = I.rng(n + len(spread))
    net = I.Network(n=n, conn="uniform", g=0.04 * 96 / n, label=spread)
    x0 = infoli.initial_state(net)
    x0[0] = SPREADS[spread](rs, n)
    small = I.Network(n=33, conn="none")
    for nets, k in (([net], 0), ([small, net], 1)):
        sim = infoli.Simulator(nets, init_states=[infoli.initial_state(m) if m is small else x0 for m in nets],
                               step_mode="graph", autotune=0)
        check_gap(sim, k, net, x0[0], o64)
        sim.close()


def test_voltage_grid_spiking_trajectory(infoli, o32, o64):
    """5,000 cells under a 25 ms pulse (every cell fires, dendrites up to tens
    of millivolts apart) for 1,000 steps with the sums ahead of the step, and
    bitwise repeatable."""
    from test_gpu_parity import check_state_bounds, compare_spikes, gpu_trace
    net = I.config2(seed=6, n=5000, pulse=True)
    net.pulses = [I.Pulse(100, 600, 6.0)]
    x0 = infoli.initial_state(net)
    got, c, t = gpu_trace(infoli, net, 1000, 100, x0, step_mode="graph", graph_chunk=50)
    again, _, _ = gpu_trace(infoli, net, 1000, 100, x0, step_mode="launch")
    np.testing.assert_array_equal(got, again)
    ref = o32.run(net, 1000, x0=x0, trace_every=100, trace_cells=net.n)
    r64 = o64.run(net, 1000, x0=x0.astype(np.float64), trace_every=100, trace_cells=net.n)
    check_state_bounds(got, ref["trace"], r64["trace"], "grid 5000")
    compare_spikes(c, t, ref["counts"], ref["times"], 64)
    assert c.min() >= 1


@pytest.mark.parametrize("n", [600, 5000])
def test_voltage_grid_keeps_a_bad_voltage_visible(infoli, n):
    """A cell whose voltage has become infinite or NaN reaches every cell's
    current, as its pair terms would."""
    net = I.Network(n=n, conn="uniform", g=0.01)
    x0 = infoli.initial_state(net)
    sim = infoli.Simulator(net, init_states=[x0], step_mode="graph", check_finite=1)
    sim.step(2)
    assert np.all(np.isfinite(sim.read_gap_current(0)))
    sim.close()
    bad = I.Network(n=n, conn="uniform", g=0.01, pulses=[I.Pulse(0, 1, 3e38, 5, 6), I.Pulse(0, 1, 3e38, 5, 6)])
    sim = infoli.Simulator(bad, init_states=[x0], step_mode="graph", check_finite=1)
    sim.step(2)
    with pytest.raises(infoli.InfoliError) as e:
        sim.sync()
    assert e.value.status == 5
    assert not np.any(np.isfinite(sim.read_gap_current(0)))
    sim.close()


def er_net(n, deg, seed, **kw):
    rp, col = I.erdos_renyi_csr(n, min(1.0, deg / max(n - 1, 1)), seed)
    rs = I.rng(seed + 1)
    return I.Network(n=n, conn="csr", g=0.04 * 96 / max(deg, 96.0), row_ptr=rp, col=col,
                     jitter=rs.uniform(-15, 15, (3, n)), **kw)


@pytest.mark.parametrize("gap", ["rgj", "sgj"])
@pytest.mark.parametrize("weights", [False, True])
@pytest.mark.parametrize("n,deg,rows", [(2, 1, 0), (255, 3, 256), (257, 40, 7), (1001, 200, 256),
                                             (1500, 1400, 8), (4099, 60, 100), (8193, 20, 256),
                                             (20001, 30, 64), (33000, 10, 32)])
def test_flat_chunked_rows(infoli, o64, n, deg, rows, weights, gap):
    """Chunked rows as flat runs (csr_path=4): rows without connections, tiles
    of one and of many chunks per thread, tile heights that are no power of
    two, the largest network staged whole and one beyond it; alone, and
    behind an odd number of cells beside all-to-all networks with and without
    the voltage grid."""
    net = er_net(n, deg, n, gap=gap)
    if weights:
        net.w_csr = (I.rng(n).uniform(0.5, 1.5, len(net.col)) * net.g).astype(np.float32)
    x0 = infoli.initial_state(net)
    sim = infoli.Simulator(net, init_states=[x0], csr_path=4, tile_rows=rows, step_mode="graph")
    assert sim.gap_path(0) == ("csr_chunked", False)
    check_gap(sim, 0, net, x0[0], o64)
    sim.close()
    others = [I.Network(n=m, conn="uniform", g=0.01, jitter=I.voltage_jitter(m, m, 15.0)) for m in (33, 600)]
    x0s = [infoli.initial_state(o) for o in others]
    sim = infoli.Simulator(others + [net], init_states=x0s + [x0], csr_path=4, tile_rows=rows, step_mode="graph")
    for k, (m, x) in enumerate(zip(others + [net], x0s + [x0])):
        check_gap(sim, k, m, x[0], o64)
    sim.step(1)
    assert np.all(np.isfinite(sim.read_state(2)))
    sim.close()


@pytest.mark.parametrize("n", [1, 2, 64, 65, 191, 192, 193, 1024, 1025, 2048])
@pytest.mark.parametrize("conn", ["uniform", "sgj", "csr", "dense", "none"])
def test_persistent_sizes(infoli, o32, o64, conn, n):
    """The persistent kernel at the sizes where its arrangement changes (a wave
    per part, split up to 192 cells, one or two cells per thread), with
    pulses, input stream and output ring: 60 steps in launches of odd lengths
    against the oracle and against one launch, bitwise."""
    from test_gpu_parity import check_state_bounds
    rs = I.rng(n + 3)
    kw = dict(jitter=rs.uniform(-10, 10, (3, n)), bias=I.input_bias(n, n), g=0.04 * 96 / max(n, 96),
              pulses=[I.Pulse(5, 30, 6.0), I.Pulse(20, 50, -2.0, 0, max(1, n // 2))])
    if conn == "csr":
        net = er_net(n, 20, n + 5)
        net.pulses, net.bias = kw["pulses"], kw["bias"]
    elif conn == "dense":
        net = I.Network(n=n, conn="dense", w_dense=rs.uniform(0, 2 * kw["g"], (n, n)).astype(np.float32), **kw)
    else:
        net = I.Network(n=n, conn="uniform" if conn == "sgj" else conn, gap="sgj" if conn == "sgj" else "rgj", **kw)
    stream = rs.normal(0.0, 1.0, (40, n)).astype(np.float32)
    x0 = infoli.initial_state(net)
    ends = []
    for lengths in ((60,), (7, 1, 52)):
        sim = infoli.Simulator(net, init_states=[x0], i_streams=[stream], step_mode="persistent", output_ring_steps=16)
        for k in lengths:
            sim.step(k)
        out = np.zeros((16, n), np.float32)
        sim.output_copy_async(44, 16, out.ctypes.data, out.size)
        sim.output_wait()
        ends.append(sim.read_state(0))
        np.testing.assert_array_equal(out[-1], ends[-1][11])
        sim.close()
    np.testing.assert_array_equal(ends[0], ends[1])
    ref = o32.run(net, 60, x0=x0, i_stream=stream)["x"]
    r64 = o64.run(net, 60, x0=x0.astype(np.float64), i_stream=stream.astype(np.float64))["x"]
    check_state_bounds(ends[0][None], ref[None], r64[None], f"persistent {conn} {n}")
