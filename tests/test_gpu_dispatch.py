"""Which kernel a call runs and the workgroup shapes it launches them in, against the oracle.

The list of candidate kernels depends on sizes and settings only, so the index of the last one
(the one without needs), which sched_status reports when no other's widths hold, says how many
were listed."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
from gpu_helpers import oracle_chains, oracle_chains_batches  # noqa: E402

from paper_2504_14966_amd.workloads import Model, Queue, random_queue  # noqa: E402

pytestmark = pytest.mark.gpu

COEF = dict(p0=2000, p1=40, d0=8000, d1=300, d2=2)
WIDE = dict(COEF, d0=1 << 24)  # a coefficient beyond the 24 bits that every static delta kernel needs


@pytest.fixture(scope="module")
def sl():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2504_14966_amd.sloanneal as m
    m.load_library()
    return m


def _selected(sl, ws):
    status = sl.sched_status(ws).cpu().tolist()
    assert status[0] == 0, status
    return status[2]


@pytest.mark.parametrize("n,B,chains", [(900, 4, 1500), (300, 1, 1500), (600, 2, 1200), (1024, 4, 2200), (700, 3, 1300)])
def test_delta_kernel_in_workgroups_of_three(sl, orc, n, B, chains):
    # the LDS holds four or five chains, and three of them spread the chains evenly
    rng = np.random.default_rng(n + B)
    q = random_queue(rng, n, max_in=100, max_out=20, thr_hi=40_000 * n)
    dq, m = sl.DeviceQueue.from_queue(q), Model(B, 0, **COEF)
    assert _selected(sl, sl.sched_anneal(dq, Model(B, 0, **WIDE), chains, 1, 0.7, 0.99, 3)) == 1
    ws = sl.sched_anneal(dq, m, chains, 60, 0.7, 0.99, 3)
    assert _selected(sl, ws) == 0
    rec, cur, best = sl.sched_chains(ws, n, chains, perms=True)
    rec, cur, best = rec.cpu().numpy(), sl.as_u16(cur), sl.as_u16(best)
    for c, (r, cu, be) in oracle_chains(q, m, [0, 1, 2, chains // 2, chains - 1], 60, 0.7, 0.99, 3, orc.start(q, m)).items():
        assert np.array_equal(rec[c], r), c
        assert np.array_equal(cur[c], cu) and np.array_equal(best[c], be), c


# (requests, fixed prefill cost, kernel that runs): the register kernel and the full replay for up to
# 64 requests; the restarted windows and the full replay above
@pytest.mark.parametrize("n,dp,selected", [(3, 4000, 0), (64, 1 << 40, 0), (3, 1 << 56, 1), (65, 4000, 0), (65, 1 << 40, 1),
                                           (130, 1 << 36, 1)])
@pytest.mark.parametrize("policy", [0, 2])
def test_fitted_candidates(sl, orc, n, dp, selected, policy):
    rng = np.random.default_rng(n + policy)
    q = random_queue(rng, n, max_in=1000, max_out=100, thr_hi=2**32 - 2)
    coef = dict(ap=3, bp=5, cp=7, dp=dp, ad=1, bd=2, cd=3, dd=11)
    fd, fo = sl.FitModel(4, policy, **coef), orc.FitModel(4, policy, **coef)
    ws = sl.sched_anneal_fit(sl.DeviceQueue.from_queue(q), fd, 5, 120, 0.5, 0.99, 3)
    assert _selected(sl, ws) == selected
    rec, cur, best = sl.sched_chains(ws, n, 5, perms=True)
    rec, cur, best = rec.cpu().numpy(), sl.as_u16(cur), sl.as_u16(best)
    info = orc.start_fit(q, fo)
    for c in range(5):
        w = orc.anneal_chain_fit(q, fo, c, 120, 0.5, 0.99, 3, start_info=info)
        assert np.array_equal(rec[c], w["rec"]), c
        assert np.array_equal(cur[c], w["cur"]) and np.array_equal(best[c], w["best"]), c


# the scale of the Metropolis test: the queue's own (0), and factors of the input order's total latency
@pytest.mark.parametrize("ratio,factor,selected", [(0, 0.0, 0), (1, 0.0, 0), (0, 1.0, 0), (1, 1.0, 0), (0, 0.03, 0),
                                                   (0, 0.02, 1), (0, 1e-4, 1), (0, 100.0, 0), (1, 3.9, 0), (1, 4.1, 1),
                                                   (1, 1e4, 1), (1, 1e-3, 0)])
def test_hot_chains_by_the_metropolis_scale(sl, orc, ratio, factor, selected):
    # 4.0 at the last proposal: four proposals per round only where that temperature is hot
    rng = np.random.default_rng(7)
    n, B, iters = 10, 4, 202
    q = random_queue(rng, n, max_in=2000, max_out=150, thr_hi=60_000 * n)
    dq, m = sl.DeviceQueue.from_queue(q), Model(B, 0, **COEF)
    m.t_ref_us = int(round(factor * orc.replay(q, m, np.arange(n, dtype=np.uint16))[1]))
    search = (ratio, 1, 0)
    ws = sl.sched_anneal(dq, m, 6, iters, 4.0, 1.0, 21, search=sl.Search(*search))
    assert _selected(sl, ws) == selected
    rec, cur, best = sl.sched_chains(ws, n, 6, perms=True)
    rec, cur, best = rec.cpu().numpy(), sl.as_u16(cur), sl.as_u16(best)
    info = orc.start(q, m, search=orc.Search(*search))
    for c, (r, cu, be) in oracle_chains(q, m, range(6), iters, 4.0, 1.0, 21, info, search).items():
        assert np.array_equal(rec[c], r), c
        assert np.array_equal(cur[c], cu) and np.array_equal(best[c], be), c


# (requests, batch, chains, candidates before the last one): two waves per chain, one, the event loop;
# above nine chains per CU the first only where one wave each would not fit at once
@pytest.mark.parametrize("n,B,chains,before", [(64, 16, 2048, 3), (64, 16, 2304, 3), (64, 16, 2305, 2), (64, 16, 3300, 2),
                                               (91, 6, 3357, 2), (200, 16, 3500, 3), (256, 32, 3000, 3)])
def test_two_proposals_per_round_by_chains(sl, orc, n, B, chains, before):
    rng = np.random.default_rng(n + chains)
    q = random_queue(rng, n, max_in=100, max_out=20, thr_hi=40_000 * n)
    dq = sl.DeviceQueue.from_queue(q)
    wide = dict(COEF, d2=1 << 25)  # no 32-bit event arithmetic: the last candidate runs
    assert _selected(sl, sl.sched_anneal(dq, Model(B, 1, t_ref_us=1, **wide), chains, 1, 0.7, 0.99, 3)) == before
    m = Model(B, 1, **COEF)
    ws = sl.sched_anneal(dq, m, chains, 40, 0.7, 0.99, 3)
    assert _selected(sl, ws) == 0
    rec, cur, best = sl.sched_chains(ws, n, chains, perms=True)
    rec, cur, best = rec.cpu().numpy(), sl.as_u16(cur), sl.as_u16(best)
    for c, (r, cu, be) in oracle_chains(q, m, [0, 5, chains // 2, chains - 1], 40, 0.7, 0.99, 3, orc.start(q, m)).items():
        assert np.array_equal(rec[c], r), c
        assert np.array_equal(cur[c], cu) and np.array_equal(best[c], be), c


# (instances, requests, chains, candidates before the full replay): mean sizes of 2 to 4
@pytest.mark.parametrize("inst,n,chains,before", [(4, 8, 256, 1), (4, 8, 257, 0), (12, 32, 200, 1), (12, 32, 929, 0),
                                                  (12, 36, 257, 0), (10, 35, 647, 0), (12, 43, 929, 1), (12, 48, 929, 1)])
def test_instances_of_a_few_requests(sl, orc, inst, n, chains, before):
    import torch
    rng = np.random.default_rng(n + chains)
    q = random_queue(rng, n, max_in=100, max_out=20, thr_hi=40_000 * n)
    where = (np.arange(n) % inst).astype(np.int32)
    dq, dw = sl.DeviceQueue.from_queue(q), torch.from_numpy(where).cuda()

    def selected(mws):
        status = sl.sched_multi_status(mws).cpu().tolist()
        assert status[0] == 0, status
        return status[2]
    wide = dict(COEF, d2=1 << 25)
    assert selected(sl.sched_anneal_multi(dq, Model(2, 1, t_ref_us=1, **wide), dw, inst, chains, 1, 0.7, 0.99, 3)) == before
    m = Model(2, 1, **COEF)
    mws = sl.sched_anneal_multi(dq, m, dw, inst, chains, 40, 0.7, 0.99, 3)
    assert selected(mws) == 0
    for k in (0, inst - 1):
        ids = np.flatnonzero(where == k)
        sub = Queue(q.in_len[ids], q.out_len[ids], q.kind[ids], q.thr_us[ids])
        rec = sl.sched_chains(mws.instance(k), len(ids), chains).cpu().numpy()
        info = orc.start(sub, m)
        for c in (0, chains // 2, chains - 1):
            assert np.array_equal(rec[c], orc.anneal_chain(sub, m, k * chains + c, 40, 0.7, 0.99, 3, start_info=info)["rec"]), (k, c)


@pytest.mark.parametrize("n,B,chains", [(70, 3, 4099), (300, 16, 5002), (1000, 8, 4201)])
@pytest.mark.parametrize("policy", [0, 2])
def test_fitted_chains_beyond_one_workgroup_per_cu(sl, orc, n, B, chains, policy):
    # workgroups of four with a ragged last one, and (1000 requests) of nine
    rng = np.random.default_rng(n + policy)
    q = random_queue(rng, n, max_in=2000, max_out=100, thr_hi=40_000_000)
    coef = dict(ap=3, bp=500, cp=20, dp=4000, ad=1, bd=70, cd=5, dd=9000)
    fd, fo = sl.FitModel(B, policy, **coef), orc.FitModel(B, policy, **coef)
    ws = sl.sched_anneal_fit(sl.DeviceQueue.from_queue(q), fd, chains, 60, 0.7, 0.99, 3)
    assert _selected(sl, ws) == 0
    rec, cur, best = sl.sched_chains(ws, n, chains, perms=True)
    rec, cur, best = rec.cpu().numpy(), sl.as_u16(cur), sl.as_u16(best)
    info = orc.start_fit(q, fo)
    for c in (0, 3, 4, chains // 2, chains - 2, chains - 1):
        w = orc.anneal_chain_fit(q, fo, c, 60, 0.7, 0.99, 3, start_info=info)
        assert np.array_equal(rec[c], w["rec"]), c
        assert np.array_equal(cur[c], w["cur"]) and np.array_equal(best[c], w["best"]), c


# Uneven workgroups: 3, 5, 6 and 7 chains each (as many as spread the chains over 256 CUs) and a
# ragged last one. (requests, batch, policy, coefficients, kernel that runs): the limit rows and the
# delta kernel of fixed-size batches, the batch-size search and list scheduling with one wave per
# chain (a timeline beyond 32 bits, where the kernel listed first does not run)
UNEVEN = {"limit_rows": (200, 20, 0, COEF, 0), "delta": (200, 3, 0, COEF, 0), "wave": (200, 40, 0, dict(COEF, d0=8_000_000), 1),
          "search": (100, 9, 2, COEF, 0), "list": (60, 7, 1, dict(COEF, d0=8_000_000), 1)}


@pytest.mark.parametrize("name", sorted(UNEVEN))
@pytest.mark.parametrize("chains", [601, 1201, 1501, 1700])
def test_uneven_workgroups(sl, orc, name, chains):
    n, B, policy, coef, selected = UNEVEN[name]
    rng = np.random.default_rng(chains + n)
    q = random_queue(rng, n, max_in=400, max_out=60, thr_hi=40_000 * n)
    m, iters = Model(B, policy, **coef), 50
    ws = sl.sched_anneal(sl.DeviceQueue.from_queue(q), m, chains, iters, 0.7, 0.99, 5)
    assert _selected(sl, ws) == selected
    waves = -(-chains // 256)
    sample = sorted({0, waves - 1, waves, chains // 2, chains // waves * waves - 1, chains - 1})
    rec, cur, best = sl.sched_chains(ws, n, chains, perms=True)
    rec, cur, best = rec.cpu().numpy(), sl.as_u16(cur), sl.as_u16(best)
    info = orc.start(q, m)
    if policy == 2:
        cs, bs, _ = sl.sched_starts(ws, n, chains)
        cs, bs = cs.cpu().numpy(), bs.cpu().numpy()
        for c, w in oracle_chains_batches(q, m, sample, iters, 0.7, 0.99, 5, info).items():
            assert np.array_equal(rec[c], w["rec"]), c
            assert np.array_equal(cur[c], w["cur"]) and np.array_equal(best[c], w["best"]), c
            assert np.array_equal(cs[c], w["cur_starts"]) and np.array_equal(bs[c], w["best_starts"]), c
        return
    for c, (r, cu, be) in oracle_chains(q, m, sample, iters, 0.7, 0.99, 5, info).items():
        assert np.array_equal(rec[c], r), c
        assert np.array_equal(cur[c], cu) and np.array_equal(best[c], be), c


@pytest.mark.parametrize("chains", [601, 1201, 1501, 1700])
def test_uneven_workgroups_fitted(sl, orc, chains):
    rng = np.random.default_rng(chains)
    n, iters, waves = 150, 60, -(-chains // 256)
    q = random_queue(rng, n, max_in=2000, max_out=100, thr_hi=40_000_000)
    coef = dict(ap=3, bp=500, cp=20, dp=4000, ad=1, bd=70, cd=5, dd=9000)
    fd, fo = sl.FitModel(6, 2, **coef), orc.FitModel(6, 2, **coef)
    ws = sl.sched_anneal_fit(sl.DeviceQueue.from_queue(q), fd, chains, iters, 0.7, 0.99, 5)
    assert _selected(sl, ws) == 0
    rec = sl.sched_chains(ws, n, chains).cpu().numpy()
    info = orc.start_fit(q, fo)
    for c in (0, waves - 1, waves, chains // 2, chains // waves * waves - 1, chains - 1):
        assert np.array_equal(rec[c], orc.anneal_chain_fit(q, fo, c, iters, 0.7, 0.99, 5, start_info=info)["rec"]), c


# (requests, batch, candidates before the full replay): limit rows and the delta kernel; one or two
# batches of up to 32 leave the limit rows out
@pytest.mark.parametrize("n,B,before", [(2, 17, 1), (30, 32, 1), (32, 32, 1), (34, 17, 1), (50, 28, 1), (64, 32, 1),
                                        (65, 32, 2), (66, 64, 2), (50, 64, 2)])
def test_two_batches_take_no_limit_rows(sl, orc, n, B, before):
    rng = np.random.default_rng(n + B)
    q = random_queue(rng, n, max_in=100, max_out=20, thr_hi=40_000 * n)
    dq, chains = sl.DeviceQueue.from_queue(q), 2600
    assert _selected(sl, sl.sched_anneal(dq, Model(B, 0, **WIDE), chains, 1, 0.7, 0.99, 3)) == before
    m = Model(B, 0, **COEF)
    ws = sl.sched_anneal(dq, m, chains, 60, 0.7, 0.99, 3)
    assert _selected(sl, ws) == 0
    rec = sl.sched_chains(ws, n, chains).cpu().numpy()
    for c, (r, _, _) in oracle_chains(q, m, [0, 7, chains - 1], 60, 0.7, 0.99, 3, orc.start(q, m)).items():
        assert np.array_equal(rec[c], r), c
