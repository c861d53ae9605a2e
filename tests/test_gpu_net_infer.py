"""Fused inference of the E network at the edges of its time tiles (250 steps
finished per tile, halos of 3 per layer), of its split over workgroups and of
both channel counts, against the oracle's emulation of the BF16 form."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import net_oracle as NO
from paper_2105_12301_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,L,B", [(64, 1, 2), (64, 7, 1), (32, 249, 2), (64, 250, 2), (64, 251, 3), (32, 256, 1),
                                   (64, 503, 1), (32, 1499, 2), (64, 2001, 2), (64, 260, 600)])
def test_fused_inference_matches_oracle(C, L, B):
    from paper_2105_12301_amd import edm

    rng = np.random.default_rng(C + L)
    theta = (synth.net_init_params(C, seed=1) + rng.normal(scale=0.05, size=edm.edm_net_param_count(C))).astype(np.float32)
    X = rng.normal(size=(B, L)).astype(np.float32)
    with edm.Context(device=0) as ctx:
        lg = edm.edm_net_forward_bf16(torch.from_numpy(theta).cuda(), C, torch.from_numpy(X).cuda(), ctx=ctx)
        ctx.sync()
    rows = np.unique(np.linspace(0, B - 1, 3).astype(int))
    ref = NO.forward_bf16(theta.astype(np.float64), X[rows], C)
    g = lg.cpu().numpy()[rows]
    # sums in FP32: a value on a BF16 rounding boundary may round the other way
    np.testing.assert_allclose(g, ref, rtol=0, atol=1e-3 * max(1.0, float(np.abs(ref).max())))
