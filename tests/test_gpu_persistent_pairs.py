"""The persistent kernel takes every ordered pair of an all-to-all network when
the caller asks for pairs (option pair_path), whatever the network's size."""
import numpy as np
import pytest

from paper_1612_01501_amd import inputs as I
from test_gpu_gap_forms import infoli  # noqa: F401
from test_gpu_parity import check_state_bounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [100, 193, 257, 600, 1024, 1025, 2048])
def test_pair_path_holds_in_the_persistent_kernel(infoli, o32, o64, n):
    rs = I.rng(n)
    net = I.Network(n=n, conn="uniform", g=0.04 * 96 / n, jitter=rs.uniform(-10, 10, (3, n)), bias=I.input_bias(n, n),
                    pulses=[I.Pulse(5, 30, 6.0)])
    x0 = infoli.initial_state(net)
    end = []
    for path in (0, 1, 2):
        sim = infoli.Simulator(net, init_states=[x0], step_mode="persistent", pair_path=path)
        sim.step(60)
        end.append(sim.read_state(0))
        sim.close()
    np.testing.assert_array_equal(end[1], end[2])       # ordered pairs both
    assert np.array_equal(end[0], end[1]) == (n <= 192)  # (the library's choice above: sums on the voltage grid)
    ref = o32.run(net, 60, x0=x0)["x"]
    r64 = o64.run(net, 60, x0=x0.astype(np.float64))["x"]
    for x in (end[0], end[1]):
        check_state_bounds(x[None], ref[None], r64[None], f"persistent {n}")
