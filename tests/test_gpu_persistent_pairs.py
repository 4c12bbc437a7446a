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


def network(kind, n, seed):
    rs = I.rng(seed)
    kw = dict(jitter=rs.uniform(-10, 10, (3, n)), bias=I.input_bias(n, seed), g=0.04 * 96 / max(n, 96),
              pulses=[I.Pulse(5, 30, 6.0), I.Pulse(20, 50, -2.0, 0, max(1, n // 2))])
    if kind == "csr":
        rp, col = I.erdos_renyi_csr(n, min(1.0, 20.0 / max(n - 1, 1)), seed)
        return I.Network(n=n, conn="csr", row_ptr=rp, col=col, **kw)
    if kind == "dense":
        return I.Network(n=n, conn="dense", w_dense=rs.uniform(0, 2 * kw["g"], (n, n)).astype(np.float32), **kw)
    return I.Network(n=n, conn="uniform" if kind == "sgj" else kind, gap="sgj" if kind == "sgj" else "rgj", **kw)


@pytest.mark.parametrize("kinds,path", [(k, 0) for k in ("csr", "dense", "none", "sgj", "csr sgj", "none sgj")] +
                         [(k, p) for k in ("uniform", "uniform csr none", "uniform dense") for p in (0, 1)])
@pytest.mark.parametrize("most,count", [(64, 300), (192, 300), (256, 300), (257, 300), (512, 600), (513, 300)])
def test_batches_past_a_network_for_each_unit(infoli, o32, o64, kinds, most, count, path):
    """More networks than compute units (256 threads each, one or two cells a
    thread; 1,024 above), of one form and of several, most of them tiny: 60 steps
    in launches of odd lengths against the oracle."""
    kinds = kinds.split()
    big = [most, most - 1, 65, 193 if most > 193 else 33]
    sizes = [big[k] if k < len(big) else 1 + k % 7 for k in range(count)]
    nets = [network(kinds[k % len(kinds)], n, k + most) for k, n in enumerate(sizes)]
    x0s = [infoli.initial_state(net) for net in nets]
    sim = infoli.Simulator(nets, init_states=x0s, step_mode="persistent", output_ring_steps=16, pair_path=path)
    for steps in (7, 1, 52):
        sim.step(steps)
    out = np.zeros((16, sum(sizes)), np.float32)
    sim.output_copy_async(44, 16, out.ctypes.data, out.size)
    sim.output_wait()
    at = np.concatenate([[0], np.cumsum(sizes)])
    for k in (0, 1, 2, 3, 4, count - 1):
        got = sim.read_state(k)
        np.testing.assert_array_equal(out[-1, at[k]:at[k + 1]], got[11])
        ref = o32.run(nets[k], 60, x0=x0s[k])["x"]
        r64 = o64.run(nets[k], 60, x0=x0s[k].astype(np.float64))["x"]
        check_state_bounds(got[None], ref[None], r64[None], f"batch {kinds} {sizes[k]}")
    sim.close()
