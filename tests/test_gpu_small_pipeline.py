"""Sweep and cross map of few series (tables and lookups of every E in one
launch each), around the rule's edges, with uneven lengths and series too short
for some or all E, against the plain form's per-E kernels."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2105_12301_amd import synth

pytestmark = pytest.mark.gpu


# N * L from one workgroup of an E to more than the one-launch form takes
@pytest.mark.parametrize("N,L,E_max,short", [(1, 200, 20, 0), (2, 64, 20, 0), (3, 300, 1, 3), (5, 1030, 20, 23), (8, 257, 7, 9),
                                             (16, 600, 8, 30), (40, 333, 20, 25), (70, 513, 5, 12), (90, 129, 20, 41)])
def test_small_pipelines_match_plain(N, L, E_max, short):
    from paper_2105_12301_amd import edm

    X, _, _ = synth.logistic_network(seed=N, N=max(N, 4), L=L)
    X = torch.from_numpy(np.ascontiguousarray(X[:N])).cuda()
    lens = np.random.default_rng(L).integers(max(2 * L // 3, 1), L + 1, size=N)
    lens[0] = L
    if short:
        lens[-1] = short  # sweep and cross map undefined from some E on
    got = {}
    for form in (edm.EDM_FORM_PLAIN, edm.EDM_FORM_CHOSEN):
        with edm.Context(device=0, form=form) as ctx:
            out = edm.edm_sweep_ccm(X, lengths=lens, E_max=E_max, ctx=ctx)
            ctx.sync()
            got[form] = [t.view(torch.int32).cpu().numpy() for t in out]
    for a, b in zip(got[edm.EDM_FORM_PLAIN], got[edm.EDM_FORM_CHOSEN]):
        assert np.array_equal(a, b)
