"""Evaluation paths that depend on the number of rows, against the oracle (bit-exact).

Candidate launches: a call whose first candidate is not the one selected, with more rows than
one pass of the grid. One order per lane: row counts that reach those kernels (checked against the
dispatch's own rule), every row against the one-order-per-wave kernels (reached by calls of few
rows) and a sample against the oracle.
"""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
from gpu_helpers import lane_shape, oracle_rows  # noqa: E402

from paper_2504_14966_amd.workloads import Model, random_queue  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sl():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2504_14966_amd.sloanneal as m
    m.load_library()
    return m


def _orders(rng, k, n):
    return rng.random((k, n)).argsort(1).astype(np.uint16)


def _spoil(p, rows, rng):
    """Rows that are no permutation: a request twice, an id of n, an id of 65535."""
    n = p.shape[1]
    for i, r in enumerate(rows):
        if i % 3 == 0 and n > 1:
            p[r, rng.integers(0, n - 1)] = p[r, n - 1]
        else:
            p[r, rng.integers(0, n)] = n if i % 3 == 1 else 65535


@pytest.mark.parametrize("d2", [3, 1 << 25])  # 64-bit times on the static kernel; the full replay
def test_later_candidate_with_many_rows(sl, orc, d2):
    rng = np.random.default_rng(d2)
    q = random_queue(rng, 12, max_in=3000, max_out=250, thr_hi=4_000_000_000)
    m = Model(5, 0, p0=5_000_000 if d2 == 3 else 2000, p1=100, d0=8_000_000 if d2 == 3 else 8000, d1=300, d2=d2,
              t_ref_us=10**6)
    p = _orders(rng, 50_000, 12)
    bad = [0, 1, 4, 8191, 8192, 32767, 32768, 49_999]
    _spoil(p, bad, rng)
    got = sl.sched_eval(sl.DeviceQueue.from_queue(q), m, sl.perms_to_device(p)).cpu().numpy()
    assert (got[bad] == -1).all()
    some = np.concatenate([np.arange(0, 50_000, 7), np.arange(49_000, 50_000)])
    assert np.array_equal(got[some], oracle_rows(q, m, p[some]))


def _layouts(rng, k, n, B):
    """k x n start flags, batch sizes uniform in 1..B."""
    out = np.zeros((k, n), np.uint8)
    at = np.zeros(k, np.int64)
    rows = np.arange(k)
    while len(rows):
        out[rows, at[rows]] = 1
        at[rows] += rng.integers(1, B + 1, len(rows))
        rows = rows[at[rows] < n]
    return out


# (n, B): one to many batches per lane, rows that straddle the 16-byte chunks of ids and flags,
# 32-position words with a remainder, and batches of the whole queue
LANES = [(2, 1), (7, 3), (10, 4), (16, 16), (33, 8), (64, 64), (100, 24), (128, 16), (200, 64)]


@pytest.mark.parametrize("n,B", LANES + [(431, 64)])  # the longest queue that fits
@pytest.mark.parametrize("rows", [65536, 65536 + 77])
def test_static_lanes(sl, orc, n, B, rows):
    assert lane_shape("static", n, B, rows)[0] == 4 and lane_shape("static", n, B, 8192)[0] == 0
    rng = np.random.default_rng(1000 * n + B + rows)
    q = random_queue(rng, n, max_in=2048, max_out=400, thr_hi=5_000_000)
    m = Model(B, 0, p0=2000, p1=40, d0=8000, d1=300, d2=2)
    p = _orders(rng, rows, n)
    bad = [0, 63, 64, 65, 127, rows // 2, rows - 64, rows - 1]
    _spoil(p, bad, rng)
    dq, dp = sl.DeviceQueue.from_queue(q), sl.perms_to_device(p)
    got = sl.sched_eval(dq, m, dp).cpu().numpy()
    assert (got[bad] == -1).all()
    # every row against the one-order-per-wave kernel (a call of few rows), a sample against the oracle
    want = np.concatenate([sl.sched_eval(dq, m, c.contiguous()).cpu().numpy() for c in dp.split(8192)])
    assert np.array_equal(got, want)
    some = rng.integers(0, rows, 256)
    assert np.array_equal(got[some], orc.eval_rows(q, m, p[some]))


@pytest.mark.parametrize("n,B", LANES + [(40, 2), (256, 64)])  # the last one the longest that fits
@pytest.mark.parametrize("rows", [16384, 16384 + 77])
def test_layout_lanes(sl, orc, n, B, rows):
    waves, _, cap = lane_shape("layout", n, B, rows)
    assert waves == 4 and lane_shape("layout", n, B, 8192)[0] == 0
    # the layouts of single requests below have more batches than a lane's entries hold, but where
    # those hold one per request
    assert (cap < n) == ((n, B) in [(33, 8), (64, 64), (100, 24), (128, 16), (200, 64), (256, 64), (16, 16)])
    rng = np.random.default_rng(1000 * n + B + rows + 1)
    q = random_queue(rng, n, max_in=2048, max_out=400, thr_hi=5_000_000)
    m = Model(B, 2, p0=2000, p1=40, d0=8000, d1=300, d2=2)
    p, s = _orders(rng, rows, n), _layouts(rng, rows, n, B)
    s[rng.integers(0, rows, 40)] = 1  # every request alone
    full = rng.integers(0, rows, 40)
    s[full] = (np.arange(n) % B == 0)
    bad = [0, 63, 64, 65, rows - 64, rows - 1]
    _spoil(p, bad, rng)
    # layouts that are not valid: no start at 0, a flag of 2 or 255, a batch one too long
    for i, r in enumerate((5, 66, 130, 4000, rows - 5)):
        if i == 0:
            s[r, 0] = 0
        elif i < 3:
            s[r, rng.integers(0, n)] = (2, 255)[i - 1]
        elif n > B:
            s[r] = (np.arange(n) % B == 0)
            at = B * rng.integers(1, (n - 1) // B + 1)
            s[r, at] = 0
        else:
            s[r, 0] = 3
        bad.append(r)
    dq, dp, ds = sl.DeviceQueue.from_queue(q), sl.perms_to_device(p), sl.starts_to_device(s)
    got = sl.sched_eval_batches(dq, m, dp, ds).cpu().numpy()
    assert (got[bad] == -1).all()
    want = np.concatenate([sl.sched_eval_batches(dq, m, a.contiguous(), b.contiguous()).cpu().numpy()
                           for a, b in zip(dp.split(8192), ds.split(8192))])
    assert np.array_equal(got, want)
    some = rng.integers(0, rows, 256)
    assert np.array_equal(got[some], orc.eval_rows_batches(q, m, p[some], s[some]))


@pytest.mark.parametrize("field,value", [("d1", (1 << 24) // 16 - 1), ("d1", (1 << 24) // 16), ("out", 5792),
                                         ("out", 5793)])
def test_static_lanes_widths(sl, orc, field, value):
    # both sides of the 24-bit factors: a full batch's sum of d1, and d2 L (L + 1) / 2 with d2 = 1
    rng = np.random.default_rng(value)
    n, B, rows = 24, 16, 32768
    assert lane_shape("static", n, B, rows)[0] == 4
    q = random_queue(rng, n, max_in=60, max_out=15, thr_hi=1_000_000_000)
    m = Model(B, 0, p0=10, p1=1, d0=10, d1=300, d2=0)
    if field == "d1":
        m.d1 = value
        q.out_len[:] = rng.integers(1, 9, n)
    else:
        m.d2 = 1
        q.out_len[3] = value
    p = _orders(rng, rows, n)
    got = sl.sched_eval(sl.DeviceQueue.from_queue(q), m, sl.perms_to_device(p)).cpu().numpy()
    some = np.arange(0, rows, 11)
    assert np.array_equal(got[some], orc.eval_rows(q, m, p[some]))


def test_lanes_unaligned_rows(sl, orc):
    # orders and flags that do not begin at a 16-byte boundary go to the one-order-per-wave kernels
    import torch
    rng = np.random.default_rng(3)
    n, B, rows = 10, 4, 40_000
    assert lane_shape("static", n, B, rows)[0] == 4 and lane_shape("layout", n, B, rows)[0] == 4
    q = random_queue(rng, n, max_in=2048, max_out=400, thr_hi=5_000_000)
    m = Model(B, 0, p0=2000, p1=40, d0=8000, d1=300, d2=2)
    p, s = _orders(rng, rows + 1, n), _layouts(rng, rows + 1, n, B)
    dq = sl.DeviceQueue.from_queue(q)
    dp = torch.from_numpy(p.view(np.int16)).cuda()[1:]
    ds = torch.from_numpy(s).cuda()[1:]
    assert dp.data_ptr() % 16 and ds.data_ptr() % 16
    some = np.arange(0, rows, 17)
    assert np.array_equal(sl.sched_eval(dq, m, dp).cpu().numpy()[some], orc.eval_rows(q, m, p[1:][some]))
    assert np.array_equal(sl.sched_eval_batches(dq, m, dp, ds).cpu().numpy()[some],
                          orc.eval_rows_batches(q, m, p[1:][some], s[1:][some]))


# (n, B): no admission, one, a ragged last part of the staged ids, one running request, every
# capacity of the list (8, 16, 32, 64 registers) full and not
CONT = [(2, 1), (9, 8), (10, 4), (20, 16), (24, 64), (50, 17), (64, 32), (97, 33), (130, 64), (400, 8)]


@pytest.mark.parametrize("n,B", CONT)
@pytest.mark.parametrize("ties", [False, True])
def test_continuous_lanes(sl, orc, n, B, ties):
    # ties: output lengths of 1 to 3, so that whole groups finish at one step (more of them than
    # the prefills at hand), with thresholds where TTFT, TPOT and end-to-end flags are mixed
    rng = np.random.default_rng(1000 * n + B + ties)
    rows = 32768 + 77
    assert lane_shape("continuous", n, B, rows)[0] > 0 and lane_shape("continuous", n, B, 4096)[0] == 0
    q = random_queue(rng, n, max_in=2048, max_out=3 if ties else 400, thr_hi=200_000 if ties else 5_000_000)
    m = Model(B, 1, p0=2000, p1=40, d0=8000, d1=300, d2=2)
    p = _orders(rng, rows, n)
    bad = [0, 63, 64, 65, 127, rows // 2, rows - 64, rows - 1]
    _spoil(p, bad, rng)
    dq, dp = sl.DeviceQueue.from_queue(q), sl.perms_to_device(p)
    got = sl.sched_eval(dq, m, dp).cpu().numpy()
    assert (got[bad] == -1).all()
    want = np.concatenate([sl.sched_eval(dq, m, c.contiguous()).cpu().numpy() for c in dp.split(4096)])
    assert np.array_equal(got, want)
    some = rng.integers(0, rows, 128)
    assert np.array_equal(got[some], orc.eval_rows(q, m, p[some]))


@pytest.mark.parametrize("field,value", [("out", 5792), ("out", 5793), ("d0", (1 << 24) - 64), ("d0", 1 << 24),
                                         ("thr", 0xFFFFFFFE), ("zero", 0)])
def test_continuous_lanes_widths(sl, orc, field, value):
    # both sides of the 24-bit factors; the largest threshold; a model whose every time is zero
    rng = np.random.default_rng(value + 5)
    n, B, rows = 20, 6, 16384
    assert lane_shape("continuous", n, B, rows)[0] > 0
    q = random_queue(rng, n, max_in=9, max_out=6, thr_hi=100_000_000)
    m = Model(B, 1, p0=10, p1=1, d0=10, d1=3, d2=1)
    if field == "out":
        q.out_len[3] = value
    elif field == "d0":
        m.d0 = value
    elif field == "thr":
        q.thr_us[::2] = value
    else:
        m = Model(B, 1, p0=0, p1=0, d0=0, d1=0, d2=0)
        q.thr_us[::2] = 0
    p = _orders(rng, rows, n)
    got = sl.sched_eval(sl.DeviceQueue.from_queue(q), m, sl.perms_to_device(p)).cpu().numpy()
    some = np.arange(0, rows, 23)
    assert np.array_equal(got[some], orc.eval_rows(q, m, p[some]))
