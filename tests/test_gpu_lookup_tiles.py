"""Lookups over every tile width (16, 8, 4, 2, 1 targets), at the edges of the
widths and of the staging's rounds, with ragged targets and any row length,
against float64 sums of the same tables."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import edm_oracle as O
from paper_2105_12301_amd import synth

pytestmark = pytest.mark.gpu
RHO_TOL = 1e-5  # as in the parity tests: float32 predictions, float64 sums


@pytest.fixture(scope="module")
def edm():
    from paper_2105_12301_amd import edm as m

    return m


# nq around one wave's queries (16), a float32 run (128), a 64-sample line, the
# widest window of each tile width (40832 / T) and the 11264 samples of a
# staging round; k over the quarters of a row; N around the tile width
@pytest.mark.parametrize("nq,k,N,E,tau,Tp", [
    (2, 1, 1, 1, 1, 0), (15, 2, 3, 2, 1, 1), (17, 3, 16, 1, 1, 0), (63, 4, 17, 3, 2, 1), (129, 5, 33, 2, 1, 0),
    (257, 6, 15, 4, 1, 3), (1000, 9, 70, 8, 1, 0), (2000, 21, 20, 20, 1, 1), (2100, 13, 1, 2, 1, 0),
    (2200, 17, 8, 16, 3, 1), (2552, 7, 17, 6, 1, 0), (2553, 8, 9, 7, 1, 1), (5104, 10, 9, 3, 1, 0),
    (5105, 3, 5, 2, 1, 0), (10208, 4, 4, 3, 1, 0), (10209, 9, 3, 2, 1, 1), (11265, 2, 5, 1, 1, 0),
    (20416, 5, 2, 4, 1, 0), (20417, 11, 2, 2, 1, 0), (32768, 1, 1, 1, 1, 0)])
def test_lookup_matches_float64(edm, nq, k, N, E, tau, Tp):
    rng = np.random.default_rng(nq + k)
    off = (E - 1) * tau + Tp
    idx = rng.integers(0, nq, size=(nq, k)).astype(np.int32)
    w = rng.random((nq, k)) + 1e-3
    w = (w / w.sum(axis=1, keepdims=True)).astype(np.float32)
    Y = (100.0 + np.cumsum(rng.standard_normal((N, nq + off)), axis=1)).astype(np.float32)
    t = off + idx.astype(np.int64)
    with edm.Context(device=0) as ctx:
        d = [torch.from_numpy(v).cuda() for v in (idx, w, Y)]
        pred, rho = edm.edm_lookup(*d, E, tau, Tp, want_pred=True, ctx=ctx)
        _, rho2 = edm.edm_lookup(*d, E, tau, Tp, want_pred=False, ctx=ctx)
        ctx.sync()
    assert torch.equal(rho.view(torch.int32), rho2.view(torch.int32))  # with and without predictions
    for j in range(N):
        y = Y[j].astype(np.float64)
        yh = (w.astype(np.float64) * y[t]).sum(axis=1)
        # weights sum to one within k * 2^-24; k + 1 roundings of values of y's size
        bound = (2 * k + 4) * 2.0 ** -24 * np.abs(y).max()
        np.testing.assert_allclose(pred[j].cpu().numpy(), yh, rtol=0, atol=bound)
        o = y[off:off + nq]
        if nq > 1 and o.std() > 0 and yh.std() > 0:
            assert abs(float(rho[j]) - np.corrcoef(o, yh)[0, 1]) <= RHO_TOL, j


# a few libraries and many, targets shorter than some libraries (undefined
# pairs) and than the offset, at the narrowest and widest tiles
@pytest.mark.parametrize("Nl,Nt,L,tau,Tp", [(1, 5, 400, 1, 0), (2, 40, 700, 1, 1), (3, 7, 300, 2, 0), (5, 130, 500, 1, 0),
                                            (9, 3, 450, 3, 1), (3, 60, 1500, 1, 0), (17, 33, 350, 1, 0), (40, 20, 200, 2, 1)])
def test_ragged_cross_maps_match_oracle(edm, Nl, Nt, L, tau, Tp):
    rng = np.random.default_rng(Nl * 100 + Nt)
    X, _, _ = synth.logistic_network(seed=2, N=max(Nl + Nt, 4), L=L)
    Lx = rng.integers(L // 2, L + 1, size=Nl)
    Ly = rng.integers(L // 2, L + 1, size=Nt)
    Ly[0], Lx[0] = L, L
    E = rng.integers(1, 9, size=Nt).astype(np.int32)
    if Nt > 5:
        Ly[-1], E[-1] = 6, 8  # shorter than its offset
    Xl, Yt = np.ascontiguousarray(X[:Nl]), np.ascontiguousarray(X[Nl:Nl + Nt])
    Yt = Yt + 50.0 * rng.random((Nt, 1)).astype(np.float32)
    ref = O.ccm(Xl, Lx, Yt, Ly, E, tau, Tp)
    got = []
    for form in (edm.EDM_FORM_CHOSEN, edm.EDM_FORM_PLAIN):
        with edm.Context(device=0, form=form) as ctx:
            rho = edm.edm_ccm(torch.from_numpy(Xl).cuda(), torch.from_numpy(E).cuda(), torch.from_numpy(Yt).cuda(), Lx=Lx, Ly=Ly,
                              tau=tau, Tp=Tp, ctx=ctx)
            ctx.sync()
            got.append(rho.cpu().numpy())
    assert np.array_equal(got[0].view(np.int32), got[1].view(np.int32))
    assert np.array_equal(np.isnan(got[0]), np.isnan(ref))
    if not np.isnan(ref).all():
        assert np.nanmax(np.abs(got[0] - ref)) <= RHO_TOL
