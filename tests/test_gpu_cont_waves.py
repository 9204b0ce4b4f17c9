"""Continuous annealing with two, four and eight proposals scored per round (the chain count picks
how many), against the oracle bit for bit: hot chains that accept nearly everything, cold ones
that accept little (the rounds then assume other outcomes), both move types, both objectives,
proposal counts that end inside a round; and several instances by the most requests one holds."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
from gpu_helpers import oracle_chains  # noqa: E402

from paper_2504_14966_amd.workloads import Model, Queue, random_queue  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sl():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2504_14966_amd.sloanneal as m
    m.load_library()
    return m


@pytest.mark.parametrize("chains", [3, 300, 600])
@pytest.mark.parametrize("n,B,T0,search,thr", [(2, 1, 1.0, None, 1 << 31), (37, 5, 50.0, None, 1 << 31),
                                               (70, 32, 1e-4, None, 0), (90, 40, 0.02, (1, 7, 0), 1 << 32),
                                               (300, 16, 0.05, None, 1 << 31)])
def test_waves_per_chain(sl, orc, chains, n, B, T0, search, thr):
    rng = np.random.default_rng(n + B)
    q = random_queue(rng, n, max_in=2000, max_out=120, thr_hi=3_000_000)
    m = Model(B, 1, p0=2000, p1=40, d0=8000, d1=300, d2=2, swap_threshold=thr)
    iters = 131
    ws = sl.sched_anneal(sl.DeviceQueue.from_queue(q), m, chains, iters, T0, 0.999, 5,
                         search=sl.Search(*search) if search else None)
    st = sl.sched_status(ws).cpu().numpy()
    assert st[0] == 0 and st[1] & 7 == 7 and st[2] == 0, st
    rec, cur, best = sl.sched_chains(ws, n, chains, perms=True)
    rec, cur, best = rec.cpu().numpy(), sl.as_u16(cur), sl.as_u16(best)
    sample = sorted({0, chains // 2, chains - 1})
    info = orc.start(q, m, search=orc.Search(*search) if search else None)
    for c, (r, cu, be) in oracle_chains(q, m, sample, iters, T0, 0.999, 5, info, search).items():
        assert np.array_equal(rec[c], r), c
        assert np.array_equal(cur[c], cu) and np.array_equal(best[c], be), c


@pytest.mark.parametrize("sizes,chains,pick", [((64, 9, 1, 0), 4, 0), ((65, 192, 3), 2, 1), ((200, 30), 3, 2),
                                               ((60, 61, 62), 200, 0)])
def test_instances(sl, orc, sizes, chains, pick):
    # LDS for at most 64 requests, at most 192, or the whole queue; more chains than fit at once
    # with eight waves each
    import torch
    rng = np.random.default_rng(sum(sizes))
    n, B, iters = sum(sizes), 7, 90
    q = random_queue(rng, n, max_in=2000, max_out=120, thr_hi=3_000_000)
    m = Model(B, 1, p0=2000, p1=40, d0=8000, d1=300, d2=2)
    inst = rng.permutation(np.repeat(np.arange(len(sizes)), sizes)).astype(np.int32)
    mws = sl.sched_anneal_multi(sl.DeviceQueue.from_queue(q), m, torch.from_numpy(inst).cuda(), len(sizes), chains,
                                iters, 0.5, 0.98, 9)
    st = sl.sched_multi_status(mws).cpu().numpy()
    assert st[0] == 0 and st[2] == pick, st
    for k, size in enumerate(sizes):
        if size == 0:
            continue
        ids = np.flatnonzero(inst == k)
        sub = Queue(q.in_len[ids], q.out_len[ids], q.kind[ids], q.thr_us[ids])
        rec, cur, best = sl.sched_chains(mws.instance(k), size, chains, perms=True)
        rec, cur, best = rec.cpu().numpy(), sl.as_u16(cur), sl.as_u16(best)
        info = orc.start(sub, m)
        for c in sorted({0, chains - 1}):
            r = orc.anneal_chain(sub, m, k * chains + c, iters, 0.5, 0.98, 9, start_info=info)
            assert np.array_equal(rec[c], r["rec"]), (k, c)
            assert np.array_equal(cur[c], r["cur"]) and np.array_equal(best[c], r["best"]), (k, c)
