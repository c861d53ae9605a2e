"""Exact scans in every workgroup layout (candidates split over waves, long
series, one-launch sweeps): tables against the oracle, and sweeps against the
two-kernel form, which shares none of the scan code.  Series of few integer
values put many equal keys in every list, so the order of ties (lower index
first) is checked across splits, lag residues and merges."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import edm_oracle as O
from paper_2105_12301_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def edm():
    from paper_2105_12301_amd import edm as m

    return m


def _series(kind, N, L, seed=5):
    if kind == "ties":
        return np.random.default_rng(seed).integers(0, 3, size=(N, L)).astype(np.float32)
    X, _, _ = synth.logistic_network(seed=seed, N=max(N, 4), L=L)
    return X[:N]


# 16 waves a query group; lengths around the 64-query groups, the 8-step blocks
# and the shortest series of each E
@pytest.mark.parametrize("kind", ["ties", "maps"])
@pytest.mark.parametrize("L,E,tau,Tp", [
    (6, 1, 1, 0), (13, 5, 1, 0), (45, 20, 1, 1), (64, 3, 1, 0), (65, 2, 1, 1), (72, 1, 1, 0),
    (129, 4, 2, 0), (200, 3, 7, 1), (257, 12, 1, 0), (300, 20, 3, 0), (1001, 7, 2, 1), (1030, 20, 1, 0)])
def test_split_tables_match_oracle(edm, kind, L, E, tau, Tp):
    x = _series(kind, 1, L)[0]
    oi, ok = O.knn(x, E, tau, Tp)
    with edm.Context(device=0) as ctx:
        idx, dist, w = edm.edm_knn(torch.from_numpy(x).cuda(), E, tau, Tp, ctx=ctx)
        ctx.sync()
    assert np.array_equal(idx.cpu().numpy(), oi)
    m = oi.shape[0]
    v = O.embed(x, E, tau)[:m].astype(np.float64)
    d = np.sqrt(((v[:, None, :] - v[oi]) ** 2).sum(axis=2))
    np.testing.assert_allclose(dist.cpu().numpy(), d, rtol=2e-7, atol=0)  # one rounding to float32 (and float64 sums)


# (series, length): 4-way splits up to 512 blocks of 256 queries, plain above;
# 16- and 8-wave workgroups above 8192 samples
@pytest.mark.parametrize("N,L,E_max,tau", [(3, 40, 20, 1), (2, 600, 20, 1), (5, 777, 6, 3), (130, 1025, 4, 1),
                                           (16, 8300, 3, 1), (16, 8300, 2, 5), (8, 19000, 2, 1)])
def test_sweep_layouts_match_two_kernel_form(edm, N, L, E_max, tau):
    X = torch.from_numpy(_series("maps", N, L)).cuda()
    lens = np.full(N, L)
    lens[-1] = max(30, L - 261)  # one shorter series
    got = {}
    for form in (edm.EDM_FORM_TWO_KERNEL, edm.EDM_FORM_PLAIN, edm.EDM_FORM_BATCHED, edm.EDM_FORM_CHOSEN):
        with edm.Context(device=0, form=form) as ctx:
            rho, E = edm.edm_simplex_sweep(X, lengths=lens, E_max=E_max, tau=tau, ctx=ctx)
            ctx.sync()
            got[form] = (rho.view(torch.int32).cpu().numpy(), E.cpu().numpy())
    ref = got[edm.EDM_FORM_TWO_KERNEL]
    for form, (rho, E) in got.items():
        assert np.array_equal(rho, ref[0]), form
        assert np.array_equal(E, ref[1]), form


# the plan's table items of long libraries cover four blocks of 256 queries
def test_plan_long_libraries_match_plain(edm):
    lens = np.array([8700, 8193, 5000, 1200, 300])
    X = torch.from_numpy(_series("ties", 5, 8700)).cuda()
    X += torch.rand(X.shape, generator=torch.Generator().manual_seed(1)).cuda() * (torch.arange(5) % 2).cuda()[:, None]
    E = np.array([1, 4, 2, 6, 3], dtype=np.int32)
    with edm.Context(device=0) as ctx:
        ref = edm.edm_ccm(X, torch.from_numpy(E).cuda(), Lx=lens, Ly=lens, ctx=ctx)
        ctx.sync()
        for form in (edm.EDM_FORM_PLAIN, edm.EDM_FORM_CHOSEN):
            ctx.set_form(form)
            plan = edm.CcmPlan(lens, lens, E, 8700, 8700, ctx=ctx)
            rho = plan.run(X, X)
            ctx.sync()
            assert torch.equal(rho.view(torch.int32), ref.view(torch.int32)), form
            plan.close()
