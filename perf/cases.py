"""The work that users of the scheduler have it do, as measurable cases.

A case names one public call (or the few calls that belong together) with its sizes:

  eval     sched_eval: score given priority orders (policy 0 static, 1 continuous admission)
  layouts  sched_eval_batches: score given orders with given batch layouts
  anneal   sched_anneal, then the winner and every chain's records and orders (policy 0
           static, 1 continuous, 2 batch sizes searched with the order: then the layouts too)
  multi    sched_assign, sched_anneal_multi and the winners of several serving instances
  fit      sched_anneal_fit: the fitted latency model with the chat SLO, and the readouts

Sizes are those of this repository's workloads, benchmark and studies, or generic. Every
output is a whole number, and every implementation of the documented rules gives the same
one, so all outputs have to agree exactly.
"""
import math

import numpy as np
import torch

import paper_2504_14966_amd.sloanneal as sl
from paper_2504_14966_amd import workloads as wl

# Queues: requests of one class (fields as the benchmark's burst queue draws them), or the
# even mix of code and chat requests with thresholds that vary by a quarter.
SINGLE, BURST, MIX = "single", "burst", "mix"


def listed():
    return [
        # a serving loop compares a handful of candidate orders of a short queue: launch latency
        {"name": "eval-few", "call": "eval", "queue": MIX, "n": 24, "B": 8, "policy": 0, "rows": 64},
        # the evaluation workload: 2^20 orders of 128 requests, static batches of 16
        {"name": "eval-static", "call": "eval", "queue": MIX, "n": 128, "B": 16, "policy": 0, "rows": 1 << 20},
        # the same orders with batch layouts of their own (the final scores of a batch-size search)
        {"name": "eval-layouts", "call": "layouts", "queue": MIX, "n": 128, "B": 16, "policy": 2, "rows": 1 << 20},
        # orders of the continuous-batching queue scored (engines that refill a slot at once)
        {"name": "eval-continuous", "call": "eval", "queue": MIX, "n": 256, "B": 32, "policy": 1, "rows": 1 << 16},
        # the paper's own scale and schedule: 10 requests, 63 levels of 100 proposals, ratio objective
        {"name": "anneal-paper", "call": "anneal", "queue": MIX, "n": 10, "B": 4, "policy": 0, "chains": 1024,
         "iters": 6300, "T0": 500.0, "alpha": 0.95, "ratio": True, "level": 100},
        # an ordinary queue of one engine: 64 requests, batches of 16
        {"name": "anneal-64", "call": "anneal", "queue": MIX, "n": 64, "B": 16, "policy": 0, "chains": 1024,
         "iters": 10000, "T0": 1.0, "alpha": 0.999},
        # a longer queue with a batch limit that is no power of two, and an odd chain count
        {"name": "anneal-ragged", "call": "anneal", "queue": SINGLE, "n": 389, "B": 24, "policy": 0, "chains": 1500,
         "iters": 4000, "T0": 1.0, "alpha": 0.9985},
        # the burst: 1024 requests at once, batches of 64 (the benchmark's headline workload)
        {"name": "anneal-burst", "call": "anneal", "queue": BURST, "n": 1024, "B": 64, "policy": 0, "chains": 4096,
         "iters": 5000, "T0": 2.0, "alpha": 0.9995},
        # the burst with the batch sizes searched as well (Algorithm 1's joint search)
        {"name": "anneal-search", "call": "anneal", "queue": BURST, "n": 1024, "B": 64, "policy": 2, "chains": 4096,
         "iters": 5000, "T0": 2.0, "alpha": 0.9995},
        # continuous admission, 32 running requests: the longest of the workloads
        {"name": "anneal-continuous", "call": "anneal", "queue": MIX, "n": 256, "B": 32, "policy": 1, "chains": 2048,
         "iters": 20000, "T0": 1.0, "alpha": 0.999},
        # Algorithm 2: the requests assigned to eight instances, every instance annealed
        {"name": "multi-8", "call": "multi", "queue": MIX, "n": 1024, "B": 16, "policy": 0, "instances": 8,
         "chains": 512, "iters": 2000, "T0": 1.0, "alpha": 0.999},
        # the fitted model (Table 2), chat and code SLOs, batch sizes searched
        {"name": "fit-search", "call": "fit", "queue": MIX, "n": 256, "B": 16, "policy": 2, "chains": 2048,
         "iters": 2000, "T0": 1.0, "alpha": 0.999},
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread evenly over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# Most request-steps (chains x proposals x requests) of a drawn annealing case, all chains
# together and in one chain, by call and policy: a drawn case then takes no longer than the
# continuous workload.
_MOST = {("anneal", 0): (8e9, 4e6), ("anneal", 1): (4e9, 2e6), ("anneal", 2): (8e9, 4e6), ("fit", 0): (2e9, 1e6),
         ("fit", 2): (2e9, 1e6), ("multi", 0): (2e9, 2e6), ("multi", 1): (2e8, 4e5)}


def draw(rng):
    call = rng.choice(["eval", "layouts", "anneal", "anneal", "anneal", "multi", "fit"])
    n, B = _log(rng, 8, 1024), _log(rng, 1, 64)
    if call in ("eval", "layouts"):
        policy = rng.choice([0, 1]) if call == "eval" else 2
        rows = _log(rng, 16, (1 << 24 if policy == 1 else 1 << 27) // max(n, 128))
        return {"call": call, "queue": rng.choice([SINGLE, MIX]), "n": n, "B": B, "policy": policy, "rows": rows}
    policy = {"anneal": rng.choice([0, 1, 2]), "multi": rng.choice([0, 1]), "fit": rng.choice([0, 2])}[call]
    c = {"call": call, "queue": MIX if call == "fit" else rng.choice([SINGLE, BURST, MIX]), "n": n, "B": B,
         "policy": policy}
    per = n
    if call == "multi":
        c["n"] = n = max(n, 32)
        c["instances"] = _log(rng, 2, 16)
        per = -(-n // c["instances"])
    total, one = _MOST[call, policy]
    c["iters"] = _log(rng, 200, max(200, min(20000, int(one / per))))
    c["chains"] = _log(rng, 1, max(1, min(4096, int(total / (n * c["iters"])))))
    c["T0"] = rng.choice([0.5, 1.0, 2.0])
    c["alpha"] = round(math.exp(-rng.uniform(2.0, 10.0) / c["iters"]), 6)  # cooled by e^-2 to e^-10 over the run
    if rng.random() < 0.25:
        c["ratio"] = True
    return c


def _queue(case, seed):
    n = case["n"]
    if case["queue"] == MIX:
        q = wl.two_class_queue(n + n % 2, seed, thr_jitter=0.25)
        return wl.Queue(q.in_len[:n], q.out_len[:n], q.kind[:n], q.thr_us[:n])
    if case["queue"] == BURST:
        return wl.single_class_queue(n, seed, in_mean=300.0, in_sd=600.0, in_hi=8192)
    return wl.single_class_queue(n, seed)


def _orders(rows, n, seed):
    """rows x n random orders (int16 holding the uint16 bits), made on the GPU in parts."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    out = torch.empty((rows, n), dtype=torch.int16, device="cuda")
    step = max(1, (1 << 25) // n)
    for r in range(0, rows, step):
        m = min(step, rows - r)
        out[r:r + m] = torch.rand((m, n), device="cuda", generator=g).argsort(1).to(torch.int16)
    return out


def _layouts(rows, n, B, seed):
    """rows x n batch-start flags with batch sizes uniform in 1..B: 256 layouts, repeated."""
    some = wl.random_layouts(np.random.default_rng(seed), min(rows, 256), n, B)
    return torch.from_numpy(some).to("cuda").repeat(-(-rows // len(some)), 1)[:rows].contiguous()


def prepare(case, seed):
    n, B, call = case["n"], case["B"], case["call"]
    st = {"case": case, "seed": int(seed)}
    if call == "fit":
        q, thr2 = wl.chat_code_queue_10ns(n + n % 2, int(seed))
        q, thr2 = wl.Queue(q.in_len[:n], q.out_len[:n], q.kind[:n], q.thr_us[:n]), thr2[:n]
        st["tpot"] = sl.thr_to_device(thr2)
        st["model"] = sl.FitModel(B, case["policy"], **sl.TABLE2_10NS)
    else:
        q = _queue(case, int(seed))
        coef = wl.MODEL_B if case["queue"] == BURST else wl.MODEL_A
        st["model"] = wl.Model(B, case["policy"], **coef)
    st["queue"] = sl.DeviceQueue.from_queue(q)
    if call in ("eval", "layouts"):
        st["orders"] = _orders(case["rows"], n, int(seed))
        st["out"] = torch.empty((case["rows"], 2), dtype=torch.int64, device="cuda")
        if call == "layouts":
            st["starts"] = _layouts(case["rows"], n, B, int(seed))
        return st
    if case.get("ratio"):
        st["search"] = sl.Search(sl.OBJ_RATIO, case.get("level", 1), 0)
    if call == "multi":
        # tokens per instance: each holds about an instance's share of the queue
        room = int(np.ceil((q.in_len.astype(np.int64) + q.out_len).sum() / case["instances"])) + 1024
        st["capacity"] = torch.full((case["instances"],), room, dtype=torch.int64, device="cuda")
        st["ws"] = sl.MultiWorkspace(n, case["instances"], case["chains"])
    else:
        st["ws"] = sl.alloc_ws(n, case["chains"])
    return st


def run(st):
    c, dq, model = st["case"], st["queue"], st["model"]
    call, n = c["call"], c["n"]
    if call == "eval":
        return sl.sched_eval(dq, model, st["orders"], out=st["out"])
    if call == "layouts":
        return sl.sched_eval_batches(dq, model, st["orders"], st["starts"], out=st["out"])
    ws, search, how = st["ws"], st.get("search"), (c["chains"], c["iters"], c["T0"], c["alpha"], st["seed"])
    if call == "multi":
        where = sl.sched_assign(dq, st["capacity"])
        sl.sched_anneal_multi(dq, model, where, c["instances"], *how, search=search, mws=ws)
        orders, keys, counts = sl.sched_multi_best(ws)
        return {"instance": where, "orders": orders, "keys": keys, "counts": counts}
    if call == "fit":
        sl.sched_anneal_fit(dq, model, *how, tpot_thr=st["tpot"], search=search, ws=ws)
    else:
        sl.sched_anneal(dq, model, *how, ws=ws, search=search)
    order, key = sl.sched_best(ws, n)
    records, final, best = sl.sched_chains(ws, n, c["chains"], perms=True)
    out = {"order": order, "key": key, "records": records, "final": final, "best": best}
    if c["policy"] == 2:
        out["final_starts"], out["best_starts"], out["starts"] = sl.sched_starts(ws, n, c["chains"])
    return out


def work(case):
    """What the call cannot do without. Bytes: the queue (9 per request) and orders read, the
    results written. Operations, in 32-bit integer ones: a scored order costs 22 per request of
    a batch whose members changed (two pair costs, the offset, the SLO test, its share of the
    sums) plus 4 per batch that only moves in time; an order scored from nothing costs a pair
    cost (3) per pair of a batch and 10 per request; continuous admission costs one insertion
    into the sorted running set (its logarithm, 2 each) and 22 per request; the fitted model
    20 per request. Annealing takes the average over its moves."""
    n, B, call, policy = case["n"], case["B"], case["call"], case["policy"]
    if call in ("eval", "layouts"):
        rows = case["rows"]
        per = n * (22 + 2 * math.log2(min(B, n) + 1)) if policy == 1 else n * (10 + 3 * min(B, n) * (0.5 if policy == 2 else 1.0))
        return {"bytes": rows * (n * (3 if call == "layouts" else 2) + 16) + 9 * n, "flops": rows * per}
    chains, m = case["chains"], n
    if call == "multi":
        chains *= case["instances"]
        m = -(-n // case["instances"])
    b = min(B, m)
    batches = -(-m // b)
    if call == "fit":
        per = 20.0 * m
    elif policy == 1:
        per = m * (22 + 2 * math.log2(b + 1)) * (2.0 / 3.0)  # from the first changed position on: two thirds on average
    elif policy == 2:
        per = 22.0 * 2 * b + 4 * batches / 2
    else:  # half the moves are swaps (two batches), half inserts (a third of the batches)
        per = (1 - 1 / batches) * (22.0 * b * (0.5 * 2 + 0.5 * (batches + 4) / 3) + 4 * batches / 3)
    state = 64 + 4 * n + (2 * n if policy == 2 else 0)
    out = 8 * case["n"] if call == "multi" else case["chains"] * state + 2 * n
    return {"bytes": 9 * n + out, "flops": chains * case["iters"] * max(per, 22.0)}


def tolerance(case):
    return "exact"


def _static_rows(q, m, order, first):
    """(met, total latency) of orders (k x n) whose batches begin where `first` is set: every
    member of a batch takes the batch's prefill, its own decode steps and, for each member j of
    the batch, j's share of the steps that both run."""
    inl, outl, kind, thr = (torch.from_numpy(np.ascontiguousarray(a).astype(np.int64)).cuda()[order] for a in
                            (q.in_len, q.out_len, q.kind, q.thr_us))
    k, n = order.shape
    pos = torch.arange(n, device="cuda")
    begin = torch.where(first, pos, 0).cummax(1).values
    wall = torch.full((k, n), n, device="cuda")
    end = torch.cat([torch.where(first, pos, wall)[:, 1:], wall[:, :1]], 1).flip(1).cummin(1).values.flip(1)
    pf = (m.p0 + m.p1 * inl).cumsum(1)
    before = torch.where(begin > 0, pf.gather(1, (begin - 1).clamp(min=0)), 0)
    prefill = pf.gather(1, end - 1) - before
    took = prefill + outl * m.d0
    for d in range(-(m.max_batch - 1), m.max_batch):
        at = pos + d
        inside = (at >= begin) & (at < end)
        at = at.clamp(0, n - 1)
        both = torch.minimum(outl, outl[:, at])
        took += torch.where(inside, both * (m.d1 + m.d2 * inl[:, at]) + m.d2 * both * (both + 1) // 2, 0)
    long = torch.zeros_like(took).scatter_reduce_(1, begin, took, "amax")  # a batch's duration at its first position
    start = (long.cumsum(1) - long).gather(1, begin)
    e2e, ttft = start + took, start + prefill
    met = torch.where(kind == 0, ttft <= thr, torch.where(kind == 1, e2e - ttft <= thr * outl, e2e <= thr))
    return torch.stack([met.sum(1), e2e.sum(1)], 1)


def _continuous_rows(q, m, order):
    """(met, total latency) of orders under continuous admission, one finish after another."""
    inl, outl, kind, thr = (torch.from_numpy(np.ascontiguousarray(a).astype(np.int64)).cuda()[order] for a in
                            (q.in_len, q.out_len, q.kind, q.thr_us))
    k, n = order.shape
    B, far = min(m.max_batch, n), 1 << 40
    left, who = torch.full((k, B), far, device="cuda"), torch.zeros((k, B), dtype=torch.int64, device="cuda")
    now, ctx, nxt = (torch.zeros(k, dtype=torch.int64, device="cuda") for _ in range(3))
    ttft, e2e = torch.zeros((k, n), dtype=torch.int64, device="cuda"), torch.zeros((k, n), dtype=torch.int64, device="cuda")
    slot = torch.arange(B, device="cuda")
    while True:
        free = left == far
        place = nxt[:, None] + free.cumsum(1) - 1  # the free slots take the next requests in order
        new = free & (place < n)
        if not bool((new | ~free).any()):
            break
        at = place.clamp(max=n - 1)
        now += torch.where(new, m.p0 + m.p1 * inl.gather(1, at), 0).sum(1)
        who = torch.where(new, at, who)
        left = torch.where(new, outl.gather(1, at), left)
        ctx += torch.where(new, inl.gather(1, at), 0).sum(1)
        ttft.scatter_add_(1, at, torch.where(new, now[:, None], 0))
        nxt += new.sum(1)
        run_ = left < far
        b, s = run_.sum(1), torch.where(run_, left, far).amin(1)
        s = torch.where(b > 0, s, 0)
        now += s * (m.d0 + m.d1 * b + m.d2 * ctx) + m.d2 * b * (s * (s + 1) // 2)
        ctx += b * s
        left = torch.where(run_, left - s[:, None], far)
        done = left == 0
        e2e.scatter_add_(1, who, torch.where(done, now[:, None], 0))
        ctx -= torch.where(done, inl.gather(1, who) + outl.gather(1, who), 0).sum(1)
        left = torch.where(done, far, left)
    met = torch.where(kind == 0, ttft <= thr, torch.where(kind == 1, e2e - ttft <= thr * outl, e2e <= thr))
    return torch.stack([met.sum(1), e2e.sum(1)], 1)


def exact(case, seed):
    """The scores of given orders in 64-bit torch; a chain's trajectory has no short form."""
    if case["call"] not in ("eval", "layouts"):
        return None
    n, B, rows = case["n"], case["B"], case["rows"]
    if rows * n * min(B, n) > 1 << 32 or (case["policy"] == 1 and rows * n * min(B, n) > 1 << 30):
        return None  # too long
    q = _queue(case, int(seed))
    m = wl.Model(B, case["policy"], **(wl.MODEL_B if case["queue"] == BURST else wl.MODEL_A))
    orders = _orders(rows, n, int(seed)).to(torch.int64) & 0xFFFF
    if case["policy"] != 1:
        first = (_layouts(rows, n, B, int(seed)) > 0 if case["call"] == "layouts" else
                 (torch.arange(n, device="cuda") % B == 0).expand(rows, n))
    out, step = [], max(1, (1 << 22) // n)
    for r in range(0, rows, step):
        part = orders[r:r + step]
        out.append(_continuous_rows(q, m, part) if case["policy"] == 1 else _static_rows(q, m, part, first[r:r + step]))
    return torch.cat(out)
