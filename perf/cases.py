"""Performance cases of the planner: what a program that plans a training iteration's memory calls, over the range of
traces it meets.

One case is one pass through the public entry points on a trace that is resident on the GPU:

  plan     load profile, B placement orders planned (first-fit, best-fit or both policies), swap scores: the step that
           a program runs once per recorded iteration to lay its pool out
  load     the load profile alone, over a time line of many iterations
  swaps    load profile, swap scores, the selection walk of all five priority scores down to a sweep of limits, the swap
           schedule of one of those selections and the replay of all of them under their limits
  weights  many weight vectors of the aggregated priority score, as one step of a tuning loop
  detect   the repeating iteration in a recorded request stream

Traces are shaped like training iterations (forward op k runs at step k, its backward at step T-1-k): weights and their
gradients live through the iteration, feature maps from their forward to their backward step, gradients two steps,
temporaries one.  Three families give the sizes: "conv" (a pyramid of feature maps), "chain" (a deep residual chain of
equal blocks, dense in long-lived variables) and "transformer" (few long-lived tensors, many one-step temporaries).
Sizes are multiples of 512 bytes and steps take 1 ms each unless the case is "timed" (0.2 to 2 ms).
"""
import math
from types import SimpleNamespace

import numpy as np
import torch
from torch.nn.functional import pad

import paper_1903_06631_amd as lap

GRANULE = 512
LINK_GBPS = 64.0
MIN_BYTES = 1 << 20
LIMITS = 21          # limits of a sweep: 0 %, 5 %, ... 100 % of the peak
LOAD_BASE = (200_000, 580)   # variables and steps of the iteration that the "load" cases repeat


def listed():
    return [
        # a small network planned while it is being built or tuned interactively: every launch counts
        dict(name="plan-conv-small", op="plan", family="conv", batch=8, px=32, vars=120, steps=22, orders=16,
             classes=False, fit="first", all=True),
        # a VGG-sized iteration, both policies tried on every second order, as the paper compares them
        dict(name="plan-conv-both-fits", op="plan", family="conv", batch=64, px=224, vars=600, steps=42, orders=256,
             classes=False, fit="both", all=False),
        # a ResNet-sized iteration with the offsets of every order asked for
        dict(name="plan-conv-large", op="plan", family="conv", batch=128, px=224, vars=3000, steps=348, orders=1024,
             classes=False, fit="first", all=True),
        # a residual chain of a few hundred blocks: odd counts, dense in long-lived variables
        dict(name="plan-chain-medium", op="plan", family="chain", batch=32, px=56, vars=9001, steps=2501, orders=193,
             classes=True, fit="first", all=False),
        # a residual chain of a thousand blocks, the densest trace there is
        dict(name="plan-chain-deep", op="plan", family="chain", batch=32, px=56, vars=50_000, steps=14_000, orders=4096,
             classes=False, fit="first", all=False),
        # a transformer's iteration planned best-fit, the paper's default policy, with a moderate number of orders
        dict(name="plan-transformer-best", op="plan", family="transformer", batch=8, px=0, vars=24_571, steps=347,
             orders=130, classes=True, fit="best", all=False),
        # a transformer's iteration with all its temporaries: the most variables
        dict(name="plan-transformer", op="plan", family="transformer", batch=8, px=0, vars=200_000, steps=580,
             orders=1024, classes=False, fit="first", all=False),
        # the load curve of a long run, iteration after iteration
        dict(name="load-iterations", op="load", family="transformer", batch=8, px=0, iterations=250),
        # swap planning for a ResNet-sized iteration with measured step times
        dict(name="swaps-conv-large", op="swaps", family="conv", batch=128, px=224, vars=3000, steps=348, timed=True),
        # swap planning for the thousand-block chain: thousands of candidates
        dict(name="swaps-chain-deep", op="swaps", family="chain", batch=32, px=56, vars=50_000, steps=14_000, timed=False),
        # one step of a tuner of the aggregated score on a transformer's iteration
        dict(name="weights-transformer", op="weights", family="transformer", batch=8, px=0, vars=200_000, steps=580,
             vectors=64, timed=False),
        # the requests of the first iterations of a large model, recorded until an iteration is seen twice
        dict(name="detect-requests", op="detect", requests=2_000_003, period=700_001),
    ]


def _between(rng, lo, hi):
    """A whole number from lo to hi, spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["plan"] * 10 + ["swaps"] * 4 + ["weights"] * 2 + ["load"] * 2 + ["detect"] * 2)
    if op == "load":
        return dict(op=op, family="transformer", batch=8, px=0, iterations=_between(rng, 1, 250))
    if op == "detect":
        m = _between(rng, 4000, 2_000_003)
        return dict(op=op, requests=m, period=int(m * rng.uniform(0.1, 0.48)))
    family = rng.choice(["conv", "chain", "transformer"])
    if family == "conv":
        n = _between(rng, 100, 6000)
        t, batch, px = max(8, int(n * rng.uniform(0.06, 0.18))), rng.choice([8, 32, 64, 100, 128]), rng.choice([32, 224])
    elif family == "chain":
        n = _between(rng, 1500, 50_000)
        t, batch, px = int(n * rng.uniform(0.2, 0.28)), rng.choice([16, 32]), 56
    else:
        n = _between(rng, 6000, 200_000)
        t, batch, px = min(580, max(48, int(n * rng.uniform(0.003, 0.02)))), 8, 0
    case = dict(op=op, family=family, batch=batch, px=px, vars=n, steps=t)
    if op == "plan":
        # best-fit looks at every hole that fits: it is for traces of mostly short lifetimes
        fit = rng.choice(["first", "first", "both", "best"]) if family == "transformer" or n <= 1000 else "first"
        most = min(4096 if n > 32_768 else 1024, 200_000_000 // n)
        if fit != "first":
            most = min(most, 512, max(16, 40_000_000 // n))
        b = _between(rng, 16, most)
        case.update(orders=b, classes=rng.random() < 0.4, fit=fit, all=bool(n * b < 10_000_000 and rng.random() < 0.5))
    elif op == "swaps":
        case.update(timed=rng.random() < 0.5)
    else:
        if family == "chain":
            case.update(vars=min(n, 12_000), steps=min(t, 3000))     # a tuner's walk over a deep chain takes seconds
        case.update(vectors=_between(rng, 4, 64), timed=rng.random() < 0.5)
    return case


# ---- inputs ----------------------------------------------------------------------------------------------------------

def _sizes(case, ops, rng):
    """Bytes of the output, parameters (0 = none), extra saved tensors (0 = none) and small saved statistics (0 = none) of every op, and a
    function that draws the sizes of temporaries."""
    k = np.arange(ops)
    zero = np.zeros(ops, np.int64)
    if case["family"] == "conv":
        stage = 5 * k // ops
        top = case["batch"] * 64 * (case["px"] // 2) ** 2 * 4
        out = np.maximum(top >> stage, GRANULE)
        weight = np.where(rng.random(ops) < 0.55, (1 << 14) << (2 * stage), 0)
        stat = np.where(rng.random(ops) < 0.3, 512 << stage, 0)
        return out, weight, zero, stat, lambda m: rng.integers(1, max(2, top // 4), m)
    if case["family"] == "chain":
        out = np.full(ops, case["batch"] * 256 * case["px"] ** 2 * 4, np.int64)
        weight = np.choose(k % 7, [256 * 256 * 36, 2048, 0, 256 * 256 * 36, 2048, 0, 0]).astype(np.int64)
        stat = np.where((k % 7 == 1) | (k % 7 == 4), 2048, 0)
        return out, weight, zero, stat, lambda m: (2.0 ** rng.uniform(12, 25, m)).astype(np.int64)
    x = case["batch"] * 2048 * 2048 * 2
    score = case["batch"] * 16 * 2048 * 2048 * 2
    layer = k % 12
    out = np.choose(layer, [x, x, score, score, x, x, x, x, 4 * x, 4 * x, x, x]).astype(np.int64)
    hid = 2048 * 2048 * 2
    weight = np.choose(layer, [8192, 3 * hid, 0, 0, 0, hid, 0, 8192, 4 * hid, 0, 4 * hid, 0]).astype(np.int64)
    extra = np.where(layer == 1, 2 * x, 0)
    stat = np.where((layer == 0) | (layer == 7), case["batch"] * 2048 * 8, 0)
    return out, weight, extra, stat, lambda m: rng.integers(1, 16 << 20, m)


def _trace(case, rng):
    """One training iteration's variables, in the order in which they are allocated."""
    n, steps = case["vars"], case["steps"]
    ops = steps // 2
    out, weight, extra, stat, temporary = _sizes(case, ops, rng)
    k = np.arange(ops)
    back = steps - 1 - k
    cols = []

    def add(size, alloc, free, lo, hi):
        size, alloc, free, lo, hi = np.broadcast_arrays(size, alloc, free, lo, hi)
        cols.append(np.stack([size, alloc, free, lo, hi]).astype(np.int64))

    idle = k + 1 <= steps - 2 - k
    lo, hi = np.where(idle, k + 1, k), np.where(idle, steps - 2 - k, steps - 1 - k)
    w = weight > 0
    add(weight[w], 0, steps, k[w], back[w])                          # parameters: read forward and backward
    add(weight[w], 0, steps, back[w], steps - 1)                     # their gradients: written backward, used at the end
    for saved in (out, extra, stat):
        s = saved > 0
        add(saved[s], k[s], steps - k[s], lo[s], hi[s])              # feature maps, saved for the backward op
    add(out, back, np.minimum(back + 2, steps), back, np.minimum(back + 1, steps - 1))    # their gradients
    used = sum(c.shape[1] for c in cols)
    assert used <= n, (used, n)
    t = rng.integers(0, steps, n - used)
    both = np.concatenate([k[w], back[w]])                           # ops with parameters use a workspace
    m = min(len(both), n - used)
    t[:m] = both[:m]
    add(temporary(n - used), t, t + 1, t, t)
    size, alloc, free, lo, hi = np.concatenate(cols, axis=1)
    order = np.argsort(alloc, kind="stable")
    size = np.maximum(GRANULE, (size + GRANULE - 1) // GRANULE * GRANULE)
    step_ns = rng.integers(200_000, 2_000_001, steps).astype(np.uint64) if case.get("timed") else None
    return SimpleNamespace(n_vars=n, n_steps=steps, size=size[order].astype(np.uint64),
                           alloc=alloc[order].astype(np.uint32), free=free[order].astype(np.uint32),
                           gap_lo=lo[order].astype(np.uint32), gap_hi=hi[order].astype(np.uint32), step_ns=step_ns)


def _iterations(tr, reps):
    """The iteration `reps` times over, one after the other."""
    shift = (np.arange(reps, dtype=np.uint32) * np.uint32(tr.n_steps))[:, None]
    return SimpleNamespace(n_vars=tr.n_vars * reps, n_steps=tr.n_steps * reps, size=np.tile(tr.size, reps),
                           alloc=(tr.alloc[None, :] + shift).reshape(-1), free=(tr.free[None, :] + shift).reshape(-1),
                           gap_lo=None, gap_hi=None, step_ns=None)


def _peak(tr):
    """The peak of the load curve and the step where it is reached first (what a program knows from its first plan)."""
    d = np.zeros(tr.n_steps + 1, np.int64)
    np.add.at(d, tr.alloc, tr.size.astype(np.int64))
    np.subtract.at(d, tr.free, tr.size.astype(np.int64))
    load = np.cumsum(d[:-1])
    return int(load.max()), int(load.argmax())


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    s = SimpleNamespace(case=case)
    if case["op"] == "detect":
        m = case["requests"]
        p = case["period"] - int(rng.integers(0, case["period"] // 3))
        # operation kind in the top byte, one of a few hundred sizes below; a warm-up that belongs to no iteration,
        # then iterations, recorded until the second one is complete
        sizes = rng.integers(1, 1 << 22, 300) * GRANULE
        tok = lambda c: (rng.integers(1, 5, c) << 56) | sizes[rng.integers(0, 300, c)]
        it = tok(p)
        stream = np.concatenate([tok(m - 2 * p), it, it])
        s.tokens = torch.from_numpy(stream.astype(np.int64)).cuda()
        s.min_period = 64
        return s
    if case["op"] == "load":
        base = _trace(dict(case, vars=LOAD_BASE[0], steps=LOAD_BASE[1]), rng)
        s.trace = lap.DeviceTrace(_iterations(base, case["iterations"]), use_gaps=False)
        return s
    tr = _trace(case, rng)
    s.trace = lap.DeviceTrace(tr)
    if case["op"] == "plan":
        b = case["orders"]
        s.kinds = np.full(b, lap.ORD_SEEDED, np.uint32)
        if case["classes"]:
            s.kinds[5::2] = lap.ORD_CLASS_SEEDED
        s.kinds[:4] = [lap.ORD_SIZE_DESC, lap.ORD_LIFE_DESC, lap.ORD_AREA_DESC, lap.ORD_ALLOC_ASC]
        s.seeds = rng.integers(0, 1 << 62, b).astype(np.uint64)
        s.fits = {"first": None, "best": [lap.FIT_BEST] * b,
                  "both": [lap.FIT_BEST if i % 2 else lap.FIT_FIRST for i in range(b)]}[case["fit"]]
        return s
    peak, at = _peak(tr)
    if case["op"] == "swaps":
        s.limits = [peak * q // (LIMITS - 1) for q in range(LIMITS)]
        return s
    s.load = lap.load_profile(s.trace)["load"]
    scores = lap.score_swaps(s.trace, LINK_GBPS, MIN_BYTES, load=s.load)
    cand = (tr.size >= MIN_BYTES) & (tr.alloc <= at) & (at < tr.free) & (tr.gap_hi > tr.gap_lo)
    s.candidates = int(cand.sum())
    sigma = [float(scores[key].cpu().numpy()[cand].astype(np.float64).std()) or 1.0 for key in ("aoa", "doa_ns", "wdoa", "wdoa")]
    s.weights = rng.uniform(-1, 1, (case["vectors"], 4)) / np.asarray(sigma)
    s.limit = peak * 6 // 10
    return s


# ---- one pass --------------------------------------------------------------------------------------------------------

def run(s):
    case = s.case
    if case["op"] == "detect":
        return lap.detect_iteration(s.tokens, s.min_period, sync=False)
    if case["op"] == "load":
        return lap.load_profile(s.trace, sync=False)
    if case["op"] == "plan":
        load = lap.load_profile(s.trace, sync=False)
        plan = lap.plan_pool(s.trace, s.kinds, s.seeds, fits=s.fits, want_all=case["all"], sync=False)
        scores = lap.score_swaps(s.trace, LINK_GBPS, MIN_BYTES, load=load["load"], sync=False)
        return dict(load=load, plan=plan, scores=scores)
    if case["op"] == "weights":
        got = lap.evaluate_weights(s.trace, LINK_GBPS, MIN_BYTES, s.weights, s.limit, load=s.load, sync=False)
        # the rows are written up to the number of candidates
        got["order"] = pad(got["order"][:, :s.candidates], (0, case["vars"] - s.candidates))
        return got
    load = lap.load_profile(s.trace, sync=False)
    scores = lap.score_swaps(s.trace, LINK_GBPS, MIN_BYTES, load=load["load"], sync=False)
    sel = lap.select_swaps(s.trace, LINK_GBPS, MIN_BYTES, [lap.PS_DOA, lap.PS_AOA, lap.PS_WDOA, lap.PS_SWDOA, lap.PS_PEAK_CUT],
                           s.limits, load=load["load"], sync=False)
    # the prefix lengths of the next calls are host values: the program reads them here
    taken = [int(x) for x in sel["n_selected"][3].tolist()]
    count = int(sel["n_cand"].item())
    order = sel["order"][3]
    schedule = lap.schedule_swaps(s.trace, LINK_GBPS, order[:taken[12]], load=load["load"], sync=False)
    replay = lap.simulate_swaps(s.trace, LINK_GBPS, order[:max(taken)], taken, s.limits, sync=False)
    # rows are written up to the number of candidates, and the orders are the inverse of the ranks; lists of varying
    # length are kept in rows of one entry per variable
    n = case["vars"]
    del sel["order"]
    sel["peaks"] = pad(sel["peaks"][:, :count + 1], (0, n - count))
    times = torch.stack([schedule.pop(key) for key in ("out_start", "out_end", "in_start", "in_end")])
    return dict(load=load, scores=scores, select=sel, times=pad(times, (0, n - taken[12])), schedule=schedule, replay=replay)


def work(case):
    """Each input read once and each output written once, and the operations that no method of placing, scoring or
    walking does without (one per variable and order, score or vector)."""
    if case["op"] == "detect":
        return dict(bytes=8 * case["requests"] + 4, flops=case["requests"])
    if case["op"] == "load":
        n, t = LOAD_BASE[0] * case["iterations"], LOAD_BASE[1] * case["iterations"]
        return dict(bytes=16 * n + 8 * t + 12, flops=2 * n + t)
    n, t = case["vars"], case["steps"]
    trace = 24 * n + (8 * t if case.get("timed") else 0)
    scores = 33 * n
    if case["op"] == "plan":
        b = case["orders"]
        return dict(bytes=trace + 8 * t + scores + 8 * n + 8 * b + (8 * b * n if case["all"] else 0), flops=n * b)
    if case["op"] == "swaps":
        return dict(bytes=trace + 8 * t + scores + 5 * 4 * n + 8 * t, flops=10 * n)
    return dict(bytes=trace + 8 * t + 8 * n, flops=n * case["vectors"])


def tolerance(case):
    return "exact"     # whole numbers throughout; the one floating score is a single operation on them
