"""Exact scans in the forms that the launch rules choose between (workgroups of 4, 8
and 16 waves, candidates queued or inserted as they come, tables of one or two E
of a group scanned alone, work lists that need few E), against forms that share
none or little of that code.  Series of few integer values put equal keys in
every list; series of huge amplitude make keys overflow to +inf."""
from __future__ import annotations

import time

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


def _series(kind, N, L, seed=7):
    r = np.random.default_rng(seed)
    if kind == "ties":
        return r.integers(0, 3, size=(N, L)).astype(np.float32)
    base = synth.logistic_network(seed=seed, N=min(max(N, 4), 8), L=L)[0]
    X = np.tile(base, (-(-N // len(base)), 1))[:N].copy()
    X *= r.uniform(0.5, 2.0, size=(N, 1)).astype(np.float32)
    if kind == "huge":
        X *= np.float32(3e19)  # about half of the keys overflow
    return X


def _sweeps(edm, forms, X, **kw):
    out = {}
    for form in forms:
        with edm.Context(device=0, form=getattr(edm, "EDM_FORM_" + form)) as ctx:
            rho, E = edm.edm_simplex_sweep(X, ctx=ctx, **kw)
            ctx.sync()
            out[form] = (rho.view(torch.int32).cpu().numpy(), E.cpu().numpy())
    return out


# (series, length, E_max, lag): more than 512 blocks of 256 queries, so nothing is
# split; as they come by 4 waves (1025), by 8 (8300 with 1024 blocks or more), by 16
# (17000); queued from E = 5 on where short
@pytest.mark.parametrize("kind,N,L,E_max,tau", [
    ("maps", 130, 1025, 8, 1), ("ties", 130, 1025, 7, 1), ("ties", 140, 1020, 6, 2), ("huge", 130, 1025, 5, 1),
    ("maps", 40, 8300, 3, 1), ("ties", 40, 8300, 2, 3), ("maps", 20, 17000, 2, 1)])
def test_sweeps_match_two_kernel_form(edm, kind, N, L, E_max, tau):
    X = torch.from_numpy(_series(kind, N, L)).cuda()
    lens = np.full(N, L)
    lens[[0, -1]] = [L - 300, L - 65]
    got = _sweeps(edm, ("TWO_KERNEL", "PLAIN", "BATCHED"), X, lengths=lens, E_max=E_max, tau=tau)
    for form in ("PLAIN", "BATCHED"):
        for a, b in zip(got["TWO_KERNEL"], got[form]):
            assert np.array_equal(a, b), form


# long series at every E: plain (one scan per E), grouped and filtered scans
@pytest.mark.parametrize("N,L", [(4, 16000), (36, 8300), (5, 32000), (30, 9000), (2, 32768)])
def test_long_sweeps_agree_between_forms(edm, N, L):
    X = torch.from_numpy(_series("maps", N, L)).cuda()
    lens = np.full(N, L)
    lens[1] = L - 4000
    got = _sweeps(edm, ("PLAIN", "BATCHED", "CHOSEN"), X, lengths=lens, E_max=20)
    for form in ("BATCHED", "CHOSEN"):
        for a, b in zip(got["PLAIN"], got[form]):
            assert np.array_equal(a, b), form


# any number of neighbours, the candidates of one series split over 16 waves
@pytest.mark.parametrize("E,k,tau,Tp,L", [(4, 1, 1, 0, 300), (3, 17, 1, 1, 257), (5, 20, 2, 0, 401), (20, 24, 1, 0, 320),
                                         (2, 31, 3, 1, 200), (1, 32, 1, 0, 65), (4, 32, 1, 0, 3000)])
def test_neighbour_counts_match_oracle(edm, E, k, tau, Tp, L):
    x = _series("ties", 1, L)[0]
    oi, _ = O.knn(x, E, tau, Tp, k=k)
    with edm.Context(device=0) as ctx:
        idx, _, w = edm.edm_knn(torch.from_numpy(x).cuda(), E, tau, Tp, k=k, ctx=ctx)
        ctx.sync()
    assert np.array_equal(idx.cpu().numpy(), oi)


# E whose tables a batched cross map needs: one or two of a group, with and without
# the few workgroups that split their candidates; and a work list of few E
@pytest.mark.parametrize("form", ["BATCHED", "CHOSEN"])
@pytest.mark.parametrize("N,L", [(3, 700), (60, 2600)])
@pytest.mark.parametrize("Es", [(1,), (2,), (5,), (9, 12), (13, 15), (18, 3), (20, 19), (1, 8), (2, 3, 8), (10, 11, 12)])
def test_cross_maps_of_few_dimensions(edm, form, N, L, Es):
    X = torch.from_numpy(_series("ties" if N == 3 else "maps", N, L)).cuda()
    E = np.array([Es[i % len(Es)] for i in range(N)], dtype=np.int32)
    lens = np.full(N, L)
    lens[1] = L - 100
    Ed = torch.from_numpy(E).cuda()
    with edm.Context(device=0) as ctx:
        ref = edm.edm_ccm(X, Ed, Lx=lens, Ly=lens, ctx=ctx)
        ctx.sync()
        ctx.set_form(getattr(edm, "EDM_FORM_" + form))
        got = edm.edm_ccm(X, Ed, Lx=lens, Ly=lens, ctx=ctx)
        plan = edm.CcmPlan(lens, lens, E, L, L, ctx=ctx)
        rho = plan.run(X, X)
        ctx.sync()
        plan.close()
    assert torch.equal(got.view(torch.int32), ref.view(torch.int32))
    assert torch.equal(rho.view(torch.int32), ref.view(torch.int32))


# keys that overflow to +inf never enter a list, in splits and merges too
@pytest.mark.parametrize("E", [1, 3, 6, 17, 20])
def test_overflowing_keys_in_splits(edm, E):
    x = torch.from_numpy(_series("huge", 1, 500)[0]).cuda()
    out = []
    for form in ("TWO_KERNEL", "PLAIN"):
        with edm.Context(device=0, form=getattr(edm, "EDM_FORM_" + form)) as ctx:
            for k in (0, E + 2):
                out.append(edm.edm_knn(x, E, 1, 0, k=k, ctx=ctx))
            ctx.sync()
    for ref, got in zip(out[:2], out[2:]):
        for a, b in zip(ref, got):
            assert torch.equal(a.view(torch.int32), b.view(torch.int32))


def test_longest_lists_of_long_series_keep_their_pace(edm):
    # 21 entries against 17: a quarter more work, and no four-way split (2.5 times
    # the time; 4.8 in workgroups of 16 waves)
    x = torch.from_numpy(_series("maps", 1, 20000)[0]).cuda()
    best = {}
    with edm.Context(device=0) as ctx:
        for E in (16, 20):
            for _ in range(6):
                t = time.perf_counter()
                edm.edm_knn(x, E, ctx=ctx)
                ctx.sync()
                best[E] = min(best.get(E, 1e9), time.perf_counter() - t)
    assert best[20] < 3.5 * best[16], best
