"""Training pass of the E network at the edges of its tiles (256 time steps a
convolution tile, 128 a gradient unit, 32 channels a matrix tile) and at channel
counts that are no multiple of a tile or of four, against the float64 oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import net_oracle as NO
from paper_2105_12301_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,L,B", [(1, 9, 2), (5, 1, 3), (16, 63, 4), (32, 128, 2), (33, 129, 3), (48, 257, 2),
                                   (64, 256, 1), (64, 521, 3), (31, 130, 40), (64, 40, 300)])
def test_loss_and_gradients(C, L, B):
    from paper_2105_12301_amd import edm

    rng = np.random.default_rng(C * 7 + L)
    theta = (synth.net_init_params(C, seed=2) + rng.normal(scale=0.05, size=edm.edm_net_param_count(C))).astype(np.float32)
    X = rng.normal(size=(B, L)).astype(np.float32)
    y = rng.integers(1, 21, size=B).astype(np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    with edm.Context(device=0) as ctx:
        loss, grad = edm.edm_net_loss_grad(dev(theta), C, dev(X), dev(y), ctx=ctx)
        logits = edm.edm_net_forward(dev(theta), C, dev(X), ctx=ctx)
        ctx.sync()
    rl, rg = NO.loss_and_grads(theta.astype(np.float64), X, y, C)
    ref, _ = NO.forward(theta.astype(np.float64), X, C)
    # float32 sums of up to 448 products a layer and 12000 (series, time) terms a gradient
    assert abs(float(loss) - rl) <= 1e-5 * max(1.0, abs(rl))
    np.testing.assert_allclose(logits.cpu().numpy(), ref, rtol=1e-4, atol=1e-5)
    np.testing.assert_allclose(grad.cpu().numpy(), rg, rtol=1e-4, atol=1e-5 * np.abs(rg).max())
