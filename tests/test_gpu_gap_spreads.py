"""All-to-all networks whose voltages leave the grid, or spread so far that a tile
takes its pairs: as near to 64 bits as sums of 32 fp32 terms added up in fp64
are, and every cell's current not finite once one voltage is not."""
import numpy as np
import pytest

from paper_1612_01501_amd import inputs as I
from test_gpu_gap_forms import infoli  # noqa: F401

pytestmark = pytest.mark.gpu

# voltages: close together but for one cell of each 64 outside the grid; over
# groups of grid points around the limits of a 64- and a 256-row tile; all of
# the grid ahead; and at its ends
SPREADS = {
    "outliers": lambda rs, n: np.where(np.arange(n) % 64 == 7, 200.0, rs.uniform(-61.0, -59.0, n)),
    "36mv": lambda rs, n: rs.uniform(-80.0, -44.1, n),
    "40mv": lambda rs, n: rs.uniform(-80.0, -39.0, n),
    "182mv": lambda rs, n: rs.uniform(-120.0, 62.0, n),
    "300mv": lambda rs, n: rs.uniform(-150.0, 150.0, n),
    "ends": lambda rs, n: np.where(rs.random(n) < 0.5, rs.uniform(-156.0, -154.0, n), rs.uniform(151.0, 155.0, n)),
}


def gauss_magnitude(v, g):
    """Per row, g times the sum over the cells of 0.8 |dV| exp(-dV^2/100)."""
    out = np.empty(len(v))
    for i in range(0, len(v), 512):
        d = np.abs(v[i:i + 512, None] - v[None, :])
        out[i:i + 512] = (0.8 * d * np.exp(-d * d / 100.0)).sum(1)
    return g * out


@pytest.mark.parametrize("spread", sorted(SPREADS))
@pytest.mark.parametrize("n", [512, 575, 1300, 4095, 4096, 5001, 16385])
def test_currents_at_any_spread(infoli, o64, n, spread):
    """Per term: the difference, its square, the exponential and the product in
    fp32, the exponent's error 2^-23 dV^2/70 of the term (16 ulp over the
    terms' range); 32 of them added one after the other; the result rounded."""
    rs = I.rng(n + len(spread))
    net = I.Network(n=n, conn="uniform", g=0.04 * 96 / n, label=spread)
    x0 = infoli.initial_state(net)
    x0[0] = SPREADS[spread](rs, n)
    vd = x0[0].astype(np.float32).astype(np.float64)
    ref = o64.gap(net, vd)
    tol = 48 * 2.0 ** -24 * gauss_magnitude(vd, net.g) + 2.0 ** -22 * np.abs(ref)
    many = [net] + [I.Network(n=64, conn="none")] * 300          # past a compute unit's 64 rows for each: 256-row tiles
    for nets in ([net], many):
        sim = infoli.Simulator(nets, init_states=[x0] + [infoli.initial_state(m) for m in nets[1:]], step_mode="graph",
                               autotune=0)
        err = np.abs(sim.read_gap_current(0).astype(np.float64) - ref) / tol
        assert err.max() <= 1.0, (len(nets), int(err.argmax()), float(err.max()))
        sim.close()


@pytest.mark.parametrize("others", [0, 300])
@pytest.mark.parametrize("n", [513, 4097])
@pytest.mark.parametrize("spread", ["outliers", "300mv"])
def test_a_bad_voltage_reaches_every_row(infoli, n, spread, others):
    net = I.Network(n=n, conn="uniform", g=0.01, pulses=[I.Pulse(0, 1, 3e38, 5, 6), I.Pulse(0, 1, 3e38, 5, 6)])
    x0 = infoli.initial_state(net)
    x0[0] = SPREADS[spread](I.rng(n), n)
    nets = [net] + [I.Network(n=64, conn="none")] * others
    sim = infoli.Simulator(nets, init_states=[x0] + [infoli.initial_state(m) for m in nets[1:]], step_mode="graph",
                           check_finite=0, autotune=0)
    assert np.all(np.isfinite(sim.read_gap_current(0)))
    sim.step(2)
    assert not np.any(np.isfinite(sim.read_gap_current(0)))
    sim.close()


@pytest.mark.parametrize("path,gap_path", [(5, ("csr_stream", True)), (1, ("csr_gather", False)), (0, None)])
def test_launches_of_large_grid_networks(infoli, o64, path, gap_path):
    """Large all-to-all networks that sum the grid themselves run in the wide
    workgroups where all networks are such, and not (but by the tuner's choice)
    where the others would need a launch beside theirs."""
    from test_gpu_gap_forms import check_gap, er_net
    csr = er_net(20000, 40, 3)
    uni = [I.Network(n=n, conn="uniform", g=0.04 * 96 / n, jitter=I.voltage_jitter(n, 5, 10.0)) for n in (5001, 4096)]
    for nets in ([csr] + uni, uni):
        x0s = [infoli.initial_state(m) for m in nets]
        sim = infoli.Simulator(nets, init_states=x0s, csr_path=path, step_mode="graph")
        info = sim.info()
        if nets is uni:
            assert info["n_tiles_wide"] == info["n_tiles"]
        elif gap_path:
            assert sim.gap_path(0) == gap_path
            assert info["n_tiles_wide"] == (79 if path == 5 else 0)
        for k, (net, x0) in enumerate(zip(nets, x0s)):
            check_gap(sim, k, net, x0[0], o64)
        sim.step(2)
        sim.sync()
        sim.close()
