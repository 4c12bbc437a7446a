"""The surrogate kernel's plain-cell lists at the sizes where they fill,
overflow and end: every cell checked every macro step takes the plain method,
so the state equals the held-gap step's bitwise, whatever the workgroup size,
the ragged last pass and the number of cells; with one cell in three checked
the unchecked cells take the MLP and the checked ones the plain result."""
import numpy as np
import pytest

from paper_1612_01501_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def infoli():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1612_01501_amd import infoli as mod
    mod.lib()
    return mod


def still_norm():
    """Inputs as they are, increments a millionth of the MLP's output."""
    return np.concatenate([np.zeros(16), np.ones(16), np.zeros(16), np.full(16, 1e-6)]).astype(np.float32)


@pytest.mark.parametrize("n", [1, 17, 64, 65, 1000, 16383, 16384, 32768, 32769, 70001])
def test_every_cell_checked_equals_the_held_gap_step(infoli, n):
    net = I.Network(n=n, conn="uniform", gap="sgj", g=0.04 * 96 / max(n, 96), jitter=I.voltage_jitter(n, n, 5.0),
                    bias=I.input_bias(n, 3), pulses=[I.Pulse(4, 9, 6.0), I.Pulse(6, 8, 1.0, 0, (n + 1) // 2)])
    x0 = infoli.initial_state(net)
    got = {}
    for mode, every in (("plain_hold", 0), ("mlp", 1), ("mlp", 3)):
        sim = infoli.Simulator(net, init_states=[x0], step_mode="launch")
        sim.surrogate_set(I.mlp_init_params(7), still_norm())
        rep = sim.step_surrogate(3, mode=mode, sample_every=every, hold_steps=0, theta_mv=1e9, z_max=0.0)
        got[every] = sim.read_state(0)
        if every:
            checked = sum(len(range((every - m % every) % every, n, every)) for m in range(3))
            assert rep["checked"] == checked and rep["plain_cell_macro_steps"] == checked
            assert rep["flagged"] == 0 and rep["guarded"] == 0
        sim.close()
    np.testing.assert_array_equal(got[1], got[0])
    # a cell checked in macro step 0 alone moved as the plain method moved it
    # there, and stood still (to the scaled output) in the other two
    moved = np.abs(got[3][1].astype(np.float64) - x0[1])
    assert np.all(np.isfinite(got[3])) and moved.max() > 0


@pytest.mark.parametrize("n,mode", [(100, "auto"), (3000, "launch"), (3000, "graph"), (9001, "graph"), (20000, "launch")])
def test_weights_replan_the_rows_and_nothing_else(infoli, n, mode):
    """Setting the weights may plan a CSR network's rows anew: the state and
    the step count stay, steps go on from there, and the
    rows' currents are the same sums (400 fp32 terms of up to 20 mV in another
    order: 400 x 2^-24 x 20 mV of each weight, ten steps of 0.05 ms)."""
    row_ptr, col = I.erdos_renyi_csr(n, min(0.3, 400.0 / n), 5)
    g = 0.04 / 400
    net = I.Network(n=n, conn="csr", row_ptr=row_ptr, col=col, g=g, bias=I.input_bias(n, 3), jitter=I.voltage_jitter(n, 4, 5.0))
    out = {}
    for weights in (False, True):
        sim = infoli.Simulator(net, init_states=[infoli.initial_state(net)], step_mode=mode, graph_chunk=2)
        sim.step(5)
        before = sim.read_state(0)
        if weights:
            sim.surrogate_set(I.mlp_init_params(7), still_norm())
            np.testing.assert_array_equal(sim.read_state(0), before)
            assert sim.last_step_ms() > 0 and sim.info()["step"] == 5
        sim.step(10)
        out[weights] = sim.read_state(0)
        sim.close()
    assert np.all(np.isfinite(out[True]))
    assert np.abs(out[True] - out[False]).max() <= 1e-3
