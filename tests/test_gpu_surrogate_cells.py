"""Each cell of a macro step takes the method its check, hold and guards give it,
and the report counts them whatever the number of workgroups and calls."""
import numpy as np
import pytest

from paper_1612_01501_amd import inputs as I
from test_gpu_gap_forms import infoli  # noqa: F401
from test_gpu_surrogate_lists import still_norm

pytestmark = pytest.mark.gpu


def sim_of(infoli, n):
    net = I.Network(n=n, conn="uniform", gap="sgj", g=0.04 * 96 / max(n, 96), jitter=I.voltage_jitter(n, n, 5.0),
                    bias=I.input_bias(n, 3))
    x0 = infoli.initial_state(net)
    return infoli.Simulator(net, init_states=[x0], step_mode="launch"), x0


@pytest.mark.parametrize("every", [2, 3, 64])
@pytest.mark.parametrize("n", [1, 17, 65, 1000, 16383, 16385, 49153, 70001])
def test_checked_cells_alone_take_the_plain_step(infoli, n, every):
    """One macro step: a checked cell as the held-gap step has it, bitwise, any
    other within the MLP's scaled increment (outputs of at most a few units, a
    millionth of them) and its rounding of where it was."""
    held, x0 = sim_of(infoli, n)
    held.step_surrogate(1, mode="plain_hold")
    plain = held.read_state(0)
    held.close()
    sim, _ = sim_of(infoli, n)
    sim.surrogate_set(I.mlp_init_params(7), still_norm())
    rep = sim.step_surrogate(1, sample_every=every, theta_mv=1e9, z_max=0.0)
    got = sim.read_state(0)
    sim.close()
    checked = np.arange(n) % every == 0
    assert rep["checked"] == rep["plain_cell_macro_steps"] == checked.sum()
    np.testing.assert_array_equal(got[:, checked], plain[:, checked])
    x0 = x0.astype(np.float32)
    still = np.abs(got.astype(np.float64) - x0) <= 1e-4 + 2.0 ** -22 * np.abs(x0)
    assert np.all(still[:, ~checked])
    if n > 1:       # the plain step moved what it should have moved
        assert np.all(np.abs(plain[0, checked] - x0[0, checked]).max() > 1e-3)


@pytest.mark.parametrize("n", [100, 16383, 16384, 70001])
def test_counts_over_calls(infoli, n):
    """Checked cells past a drift bound of zero are held for two macro steps; calls
    of one, three and two macro steps, with and without a report."""
    sim, _ = sim_of(infoli, n)
    sim.surrogate_set(I.mlp_init_params(7), still_norm())
    hold = np.zeros(n, int)
    m = 0
    for calls, report in ((1, True), (3, True), (1, False), (2, True)):
        want = np.zeros(4, int)
        for _ in range(calls):
            check = (np.arange(n) + m) % 5 == 0
            plain = check | (hold > 0)
            hold = np.where(check, 2, np.maximum(hold - plain, 0))
            want += [plain.sum(), check.sum(), check.sum(), 0]
            m += 1
        rep = sim.step_surrogate(calls, sample_every=5, theta_mv=0.0, hold_steps=2, z_max=0.0, report=report)
        if report:
            assert [rep[k] for k in ("plain_cell_macro_steps", "checked", "flagged", "guarded")] == list(want)
    sim.close()
