"""The surrogate's own gap launch: setting the weights leaves the plain steps as
they were planned, the macro steps do not depend on the shapes the tuner chose,
and every shape the rule takes gives the network's gap currents."""
import numpy as np
import pytest

from paper_1612_01501_amd import inputs as I
from test_gpu_gap_forms import er_net, infoli  # noqa: F401
from test_gpu_parity import gap_bound
from test_gpu_surrogate_lists import still_norm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,deg,kw", [(300, 20, {}), (3000, 400, {}), (9001, 60, {}), (20000, 120, {}),
                                      (3000, 60, dict(csr_path=4)), (3000, 60, dict(autotune=0, step_mode="graph"))])
def test_weights_leave_the_plain_steps_alone(infoli, n, deg, kw):
    """Same plan, same bits: five steps, the weights, eleven more."""
    net = er_net(n, deg, 5)
    x0 = infoli.initial_state(net)
    sim = infoli.Simulator(net, init_states=[x0], **kw)
    sim.step(5)
    mid, plan = sim.read_state(0), (sim.gap_path(0), sim.info())
    sim.step(11)
    end = sim.read_state(0)
    sim.write_state(0, mid, 5)
    ms = sim.last_step_ms()
    sim.surrogate_set(I.mlp_init_params(7), still_norm())
    np.testing.assert_array_equal(sim.read_state(0), mid)
    info = sim.info()
    assert sim.gap_path(0) == plan[0] and info["step"] == 5 and sim.last_step_ms() == pytest.approx(ms, rel=1e-3)
    for k in ("tuned", "tune_cached", "tune_mode", "n_tiles", "tile_rows", "lanes_per_row", "n_blocked", "n_stream", "n_bitmap"):
        assert info[k] == plan[1][k], k
    sim.step(11)
    np.testing.assert_array_equal(sim.read_state(0), end)
    sim.close()


@pytest.mark.parametrize("n,deg", [(1000, 150), (4100, 60), (9001, 150), (20000, 120)])
def test_macro_steps_do_not_follow_the_tuner(infoli, n, deg, tmp_path, monkeypatch):
    """The same macro steps whatever shapes the tuner's cache holds: as timed,
    and with every shape replaced by other lane groups or other rows."""
    net = er_net(n, deg, 7)
    x0 = infoli.initial_state(net)
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("INFOLI_TUNE_CACHE", str(cache))
    got = []
    for shape in (None, "32 8 0 0 256 8192", "4 64 0 3 256 8192"):
        if shape:
            lines = [ln.split("|") for ln in cache.read_text().splitlines()]
            cache.write_text("".join(f"{k}|{v if k.startswith('ctx ') else shape if '#256nc' not in k else '32 8 0 0 256 8192'}\n"
                                     for k, v in lines if "#bm" not in k))
        sim = infoli.Simulator(net, init_states=[x0], step_mode="launch")
        sim.surrogate_set(I.mlp_init_params(7), still_norm())
        sim.step_surrogate(5, sample_every=3, theta_mv=1e9, z_max=0.0)
        got.append(sim.read_state(0))
        sim.close()
    np.testing.assert_array_equal(got[1], got[0])
    np.testing.assert_array_equal(got[2], got[0])


@pytest.mark.parametrize("n,deg,kind", [
    (5, 2, "rgj"), (300, 20, "rgj"), (1000, 150, "rgj"), (1000, 200, "sgj"), (1001, 500, "rgj"), (4099, 1300, "rgj"),
    (8192, 60, "rgj"), (9001, 60, "weights"), (9001, 420, "rgj"), (9001, 420, "weights"), (20001, 60, "rgj"),
    (20001, 100, "rgj"), (20001, 100, "weights"), (32768, 50, "sgj"), (32769, 50, "rgj")])
def test_held_gap_currents_of_every_shape(infoli, o64, n, deg, kind):
    """One held-gap macro step against the same from the oracle's gap currents:
    the first cell voltage after four steps of 0.05 ms with a current held, so
    0.2 times its bound, times at most four for the total conductance (below
    8 mS, 1.4^4), and an fp32 ulp of the voltage a step."""
    net = er_net(n, deg, n, gap="sgj" if kind == "sgj" else "rgj")
    if kind == "weights":
        net.w_csr = (I.rng(n).uniform(0.5, 1.5, len(net.col)) * net.g).astype(np.float32)
    x0 = infoli.initial_state(net)
    sim = infoli.Simulator(net, init_states=[x0], step_mode="launch")
    sim.step_surrogate(1, mode="plain_hold")
    got = sim.read_state(0)
    sim.close()
    gap = o64.gap(net, x0[0].astype(np.float64))
    # the oracle's four steps of uncoupled cells with the current as a negative bias
    alone = I.Network(n=n, conn="none", bias=(-gap).astype(np.float32))
    ref = o64.run(alone, 4, x0=x0.astype(np.float64))["x"]
    tol = 4 * 0.2 * gap_bound(net, x0[0]) + 16 * 2.0 ** -24 * np.abs(x0[0]).max() + 0.8 * 2.0 ** -24 * np.abs(gap)
    err = np.abs(got[0].astype(np.float64) - ref[0]) / tol
    assert err.max() <= 1.0, (int(err.argmax()), float(err.max()))
