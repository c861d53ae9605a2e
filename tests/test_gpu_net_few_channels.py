"""The E network with few channels (one block of 8, far less than a matrix tile
of 32) over many slices of a gradient, and with channel counts just above a
block, against the float64 oracle; and the time of such a pass, which must not
grow as the channels shrink (a gradient reduced by one wave took 22 times as
long at one channel as at sixteen)."""
from __future__ import annotations

import time

import numpy as np
import pytest
import torch

from oracle import net_oracle as NO
from paper_2105_12301_amd import edm, synth

pytestmark = pytest.mark.gpu


def _case(C, L, B):
    rng = np.random.default_rng(C * 11 + L)
    theta = (synth.net_init_params(C, seed=3) + rng.normal(scale=0.05, size=edm.edm_net_param_count(C))).astype(np.float32)
    return theta, rng.normal(size=(B, L)).astype(np.float32), rng.integers(1, 21, size=B).astype(np.int32)


def _dev(a):
    return torch.from_numpy(a).cuda()


@pytest.mark.parametrize("C,L,B", [(1, 700, 9), (2, 1, 5), (3, 300, 6), (7, 129, 4), (8, 900, 5), (9, 513, 4),
                                   (17, 260, 3), (25, 131, 4), (40, 300, 3), (41, 127, 2), (57, 255, 2)])
def test_loss_gradients_and_logits(C, L, B):
    theta, X, y = _case(C, L, B)
    with edm.Context(device=0) as ctx:
        loss, grad = edm.edm_net_loss_grad(_dev(theta), C, _dev(X), _dev(y), ctx=ctx)
        logits = edm.edm_net_forward(_dev(theta), C, _dev(X), ctx=ctx)
        ctx.sync()
    rl, rg = NO.loss_and_grads(theta.astype(np.float64), X, y, C)
    ref, _ = NO.forward(theta.astype(np.float64), X, C)
    # float32 sums of up to 399 products a layer and 6300 (series, time) terms a gradient
    assert abs(float(loss) - rl) <= 1e-5 * max(1.0, abs(rl))
    np.testing.assert_allclose(logits.cpu().numpy(), ref, rtol=1e-4, atol=1e-5)
    np.testing.assert_allclose(grad.cpu().numpy(), rg, rtol=1e-4, atol=1e-5 * np.abs(rg).max())


@pytest.mark.parametrize("C,L,B", [(32, 8, 40), (64, 8, 40), (64, 33, 5), (32, 282, 3), (64, 282, 3)])
def test_short_and_last_tiles_of_the_inference(C, L, B):
    theta, X, _ = _case(C, L, B)
    with edm.Context(device=0) as ctx:
        lg = edm.edm_net_forward_bf16(_dev(theta), C, _dev(X), ctx=ctx)
        ctx.sync()
    ref = NO.forward_bf16(theta.astype(np.float64), X, C)
    # sums in FP32: a value on a BF16 rounding boundary may round the other way
    np.testing.assert_allclose(lg.cpu().numpy(), ref, rtol=0, atol=1e-3 * max(1.0, float(np.abs(ref).max())))


def test_one_channel_takes_no_longer_than_sixteen():
    best = {}
    with edm.Context(device=0) as ctx:
        for C in (1, 16):
            theta, X, y = (_dev(a) for a in _case(C, 1500, 64))
            for _ in range(12):
                t = time.perf_counter()
                edm.edm_net_loss_grad(theta, C, X, y, ctx=ctx)
                ctx.sync()
                best[C] = min(best.get(C, 1e9), time.perf_counter() - t)
    assert best[1] < 2 * best[16], best
