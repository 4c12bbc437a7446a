"""The gradient kernels at the edges of their split: fewer groups of 16 samples
than slices of the batch, slices of unequal length, more groups than
workgroups, and batches whose tiles are shared by several workgroups."""
import numpy as np
import pytest

from oracle import mlp as M
from paper_1612_01501_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def infoli():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1612_01501_amd import infoli as mod
    mod.lib()
    return mod


@pytest.mark.parametrize("batch", [16, 48, 272, 2064, 8208, 12272, 12288, 33040])
def test_gradients_over_the_splits(infoli, batch):
    """Against the emulated-BF16 oracle: a BF16 rounding that fp32 and fp64 sums
    send different ways moves an element by about 1e-4 of its block's largest
    at 64 samples (one activation's last bit, one term of the sum), by 64/batch
    of that elsewhere; ten times that for smaller batches, and the 1e-3 of 64
    samples for larger ones, where fp32 sums add 2^-24 sqrt(batch)."""
    w = I.mlp_init_params(5)
    w = w + np.random.default_rng(6).normal(0.0, 0.02, w.shape).astype(np.float32)
    x, t = I.mlp_batch(batch, batch)
    loss, g = infoli.mlp_loss_grad(w, x, t)
    rl, rg = M.loss_and_grad(w.astype(np.float64), x, t, bf16=True)
    tol = 1e-3 * max(1.0, 64.0 / batch)
    assert loss == pytest.approx(rl, rel=1e-4)
    gp, rp = M.unpack(g.astype(np.float64)), M.unpack(rg)
    for name, _ in M.SHAPES:
        a, b = gp[name], rp[name]
        if name in ("W3", "b3"):                    # rows 14, 15 are padding outputs
            assert np.all(a[14:] == 0), name
            a, b = a[:14], b[:14]
        assert np.all(np.abs(a - b) <= tol * np.abs(b).max()), name
        assert np.linalg.norm(a - b) <= tol * np.linalg.norm(b), name
