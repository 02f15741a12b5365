"""Measured cases of the memory planner: the calls a program makes, over the
sizes, orders and options it makes them with.

A case is a dict of plain values: the entry point (`op`), the shape of its
traces (`kind`), how many and how long they are, the order of the tensors
(`recorded`: by first op, as an allocation recorder lists them; `shuffled`: any
order) and the sizes' unit (64: an allocator's rounding; 4: raw sizes of 32-bit
elements; 1: of bytes).
Every pass goes through the Python entry points as a serving loop uses them:
buffers, workspace and the sticky status word are kept by the caller and the
status is looked at later, not after every call.  The status word is among the
outputs, so a pass that raised a code shows.

All outputs are whole numbers and every one is determined by the inputs, so
they have to be the same, not close.  The one exception is the optimum's
offsets, where several plans reach the same peak: there the peaks and the
number of conflicting pairs of the plan (from the batch validation, as a
program would check it) are returned.
"""
import math

import numpy as np
import torch

from paper_2203_00448_amd import binding

BATCH_MAX = binding.BATCH_MAX_TRACE_LEN
ARENA = 64 << 20  # bytes: above the peak of every probed plan
POLICIES = {"lowest": binding.LOWEST_FIT, "best": binding.BEST_FIT}


def listed():
    def case(name, op, kind, n, traces=1, policy="lowest", order="recorded", unit=64):
        return {"name": name, "op": op, "kind": kind, "n": n, "traces": traces, "policy": policy,
                "order": order, "unit": unit}

    return [
        # one small model planned on its own: launches and latency only
        case("trace_chain256", "trace", "chain", 256),
        # one CNN, listed in any order with raw sizes, tightest gap
        case("trace_cnn_best", "trace", "resnext", 3001, policy="best", order="shuffled", unit=4),
        # a long decode loop: long chains of equal sizes, some tensors living to the end
        case("trace_decode100k", "trace", "decode", 100_000),
        # a ranking model: thousands of tensors alive at once
        case("trace_ranking1m", "trace", "ranking", 1_000_000),
        # the benchmark's step: a large batch planned, then its plan checked
        case("step_resnext_batch", "step", "resnext", 2000, traces=1024),
        # a handful of small models at once
        case("batch_few", "batch", "resnext", 700, traces=12),
        # a mixed batch: ragged lengths up to the longest accepted, any order, raw sizes, tightest gap
        case("batch_ragged_best", "batch", "resnext", 4096, traces=600, policy="best",
             order="shuffled", unit=4),
        # a plan that somebody edited, checked: the exact list of conflicting pairs
        case("validate_decode100k", "validate", "decode", 100_000),
        # the same plan replayed over its slab
        case("probe_decode100k", "probe", "decode", 100_000),
        # the baseline figures of a long trace: live bytes per op, and the arena without reuse
        case("live_bump_ranking1m", "live_bump", "ranking", 1_000_000),
        # the other greedy strategy over the benchmark's batch
        case("breadth_resnext_batch", "breadth", "resnext", 2000, traces=1024),
        # the exact optimum of many tiny traces
        case("optimal_tiny", "optimal", "tiny", 10, traces=2048),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case.  `n` is a trace's length, in a batch the longest: the
    others are spread below it.  The bounds keep a pass below the million
    tensor trace's."""
    op = rng.choice(["trace", "trace", "trace", "batch", "batch", "step", "validate", "probe",
                     "live_bump", "breadth", "optimal"])
    order = rng.choice(["recorded", "recorded", "shuffled"])
    unit = rng.choice([64, 64, 4, 1])
    policy = rng.choice(["lowest", "lowest", "best"])
    traces = 1
    if op == "trace":
        kind = rng.choice(["chain", "resnext", "decode", "ranking"])
        top = {"chain": 30_000, "resnext": 30_000, "decode": 100_000, "ranking": 300_000}[kind]
        if policy == "best":
            top = min(top, 20_000 if kind in ("chain", "resnext") else 8_000)
        n = _log_int(rng, 64, top)
    elif op in ("batch", "step"):
        kind = rng.choice(["chain", "resnext", "resnext"])
        traces, n = _log_int(rng, 1, 1024), _log_int(rng, 64, BATCH_MAX)
        if op == "step":
            order, policy = "recorded", "lowest"
    elif op in ("validate", "probe"):
        kind = rng.choice(["resnext", "decode", "ranking"])
        n, policy, unit = _log_int(rng, 256, 60_000), "lowest", 64
        if op == "probe":
            kind = rng.choice(["decode", "ranking"])
    elif op == "live_bump":
        kind = rng.choice(["decode", "ranking", "resnext"])
        n, policy = _log_int(rng, 256, 1_000_000), "lowest"
    elif op == "breadth":
        kind = "resnext"
        traces, n = _log_int(rng, 1, 1024), _log_int(rng, 64, binding.BREADTH_MAX_TRACE_LEN)
    else:
        kind, policy = "tiny", "lowest"
        traces, n = _log_int(rng, 16, 2048), rng.randint(4, 10)
    return {"op": op, "kind": kind, "n": n, "traces": traces, "policy": policy, "order": order,
            "unit": unit}


def _traces(kind, n, rng):
    """Births, deaths and sizes (before rounding) of a trace of n tensors in
    recorded order, and its op count.  The shapes are those of
    paper_2203_00448_amd.tracegen, for any length."""
    i = np.arange(n, dtype=np.int64)
    if kind == "chain":         # one birth per op, dead a few ops later, 1 KiB .. 4 MiB
        ops, first = n, i
        last = first + 1 + (rng.geometric(0.5, n) - 1)
        size = 2.0 ** rng.uniform(10, 22, n)
    elif kind == "resnext":     # one birth per op, a tenth of them skip connections
        ops, first = n, i
        skip = rng.random(n) < 0.10
        last = first + np.where(skip, rng.integers(10, 51, n), rng.integers(1, 4, n))
        size = np.clip(np.exp(np.log(819200.0) + 1.2 * rng.standard_normal(n)), 4096, 2.0 ** 26)
    elif kind == "tiny":        # the same in miniature
        ops, first = n, i
        skip = rng.random(n) < 0.20
        last = first + np.where(skip, rng.integers(2, max(2, n // 2) + 1, n),
                                rng.integers(1, 3, n))
        size = np.clip(np.exp(np.log(819200.0) + 1.2 * rng.standard_normal(n)), 4096, 2.0 ** 26)
    elif kind == "decode":      # 25 births per op, short lives, 2% live to the end
        ops, first = (n + 24) // 25, i // 25
        last = first + rng.geometric(0.3, n) - 1
        last = np.where(rng.random(n) < 0.02, ops - 1, last)
        size = np.minimum(256.0 * (1.0 - rng.random(n)) ** (-1.0 / 1.5), 2.0 ** 28)
    elif kind == "ranking":     # ten births per op, lives of up to a thousand ops
        ops, first = (n + 9) // 10, i // 10
        last = first + rng.integers(1, 1001, n)
        size = 2.0 ** (6.0 + 10.0 * rng.random(n))
    else:
        raise ValueError(kind)
    return first, np.minimum(last, ops - 1), np.floor(size).astype(np.int64), ops


def _lengths(case):
    """Trace lengths of a batch: all `n` for the benchmark's batch and the tiny
    traces, otherwise spread from a thirty-second of n up to n, one of them n
    (a program's set of models: the same for every seed)."""
    n, k = case["n"], case["traces"]
    rng = np.random.default_rng([n, k])
    if case["op"] in ("step", "breadth", "optimal"):
        return np.full(k, n)
    low = max(1, n // 32)
    out = np.exp(rng.uniform(np.log(low), np.log(n), k)).round().astype(np.int64)
    out[0] = n
    return out


def _bound(case):
    """The bound a program states for its batches: its longest trace rounded up
    to a whole number of 64s (512 at least where the order is arbitrary)."""
    least = 512 if case["order"] == "shuffled" else 64
    return min(BATCH_MAX, max(least, (case["n"] + 63) // 64 * 64))


def _inputs(case, seed):
    """(begin, num_ops, size, first, last) as numpy arrays."""
    rng = np.random.default_rng([int(seed), 17])
    lengths = _lengths(case) if case["traces"] > 1 else np.array([case["n"]])
    parts, ops = [], []
    for length in lengths:
        first, last, size, n_ops = _traces(case["kind"], int(length), rng)
        if case["order"] == "shuffled":
            p = rng.permutation(int(length))
            first, last, size = first[p], last[p], size[p]
        parts.append((size, first, last))
        ops.append(n_ops)
    size, first, last = (np.concatenate(a) for a in zip(*parts))
    unit = case["unit"]
    size = (np.maximum(size, 1) + unit - 1) // unit * unit
    begin = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    return begin, np.asarray(ops, np.int32), size, first.astype(np.int32), last.astype(np.int32)


def _edit(offset, seed):
    """A plan with one tensor in a thousand (at least one) moved onto its neighbour in the list."""
    n = offset.numel()
    rng = np.random.default_rng([int(seed), 23])
    ids = np.unique(rng.integers(0, n - 1, max(1, n // 1000)))
    to = torch.from_numpy(ids).to(offset.device)
    out = offset.clone()
    out[to] = offset[to + 1]
    return out


def prepare(case, seed):
    begin, ops, size, first, last = _inputs(case, seed)
    dev = "cuda"
    n, k = len(size), len(ops)
    s = {"case": case, "begin": torch.from_numpy(begin).to(dev),
         "ops": torch.from_numpy(ops).to(dev), "size": torch.from_numpy(size).to(dev),
         "first": torch.from_numpy(first).to(dev), "last": torch.from_numpy(last).to(dev),
         "num_ops": int(ops.max()), "policy": POLICIES[case["policy"]], "bound": _bound(case),
         "status": binding.new_status(dev)}

    def buf(count, dtype=torch.int64):
        return torch.zeros(count, dtype=dtype, device=dev)

    def work(op, *a):
        return buf(max(1, binding.workspace_size(op, *a)), torch.uint8)

    trace = (s["size"], s["first"], s["last"])
    op = case["op"]
    s["out"] = (buf(n), buf(k)) if op != "live_bump" else None
    if op in ("trace", "validate", "probe"):
        s["ws"] = work(binding.OP_PLAN_TRACE, n, s["num_ops"])
    if op in ("batch", "step"):
        s["out"] += (buf(k),)
        s["ws"] = work(binding.OP_PLAN_BATCH, n, k)
    if op in ("step", "optimal"):
        s["cap"] = 4096
        s["pairs"] = (buf((s["cap"], 2)), buf(1))
        s["vws"] = work(binding.OP_VALIDATE_BATCH, n, k, s["cap"])
    if op in ("validate", "probe"):
        off, peak = binding.plan_trace(*trace, s["num_ops"], out=s["out"], workspace=s["ws"])
        s["plan"] = _edit(off, seed) if op == "validate" else off.clone()
        if op == "validate":
            s["cap"] = 1 << 20  # the entry point's own default
            s["pairs"] = (buf((s["cap"], 2)), buf(1))
            s["ws"] = work(binding.OP_VALIDATE, n, 0, s["cap"])
        else:
            # the plan's bytes at the front of the arena that the program keeps
            s["arena"] = torch.full((ARENA,), 0xA5, dtype=torch.uint8, device=dev)
            s["slab"] = s["arena"][:int(peak.item())]
            s["out"] = (buf(n, torch.uint8), buf(1))
            s["ws"] = work(binding.OP_PROBE, n, s["num_ops"])
    if op == "live_bump":
        s["live"] = (buf(s["num_ops"]), buf(1))
        s["bump"] = (buf(n), buf(1))
        s["ws"] = work(binding.OP_LIVE_BYTES, n, s["num_ops"])
        s["bws"] = work(binding.OP_BUMP, n)
    return s


def run(s):
    op, st = s["case"]["op"], s["status"]
    trace = (s["size"], s["first"], s["last"])
    if op == "trace":
        out = binding.plan_trace(*trace, s["num_ops"], policy=s["policy"], check=False,
                                 out=s["out"], status=st, workspace=s["ws"])
        return out, st
    if op in ("batch", "step"):
        out = binding.plan_batch(s["begin"], s["ops"], *trace, max_trace_len=s["bound"],
                                 policy=s["policy"], check=False, out=s["out"], status=st,
                                 workspace=s["ws"])
        if op == "batch":
            return out, st
        pairs, count, _ = binding.validate_batch(
            s["begin"], *trace, out[0], capacity=s["cap"], check=False, status=st,
            workspace=s["vws"], out=s["pairs"], assume_sorted=True, max_trace_len=s["bound"])
        return out, pairs, count, st
    if op == "validate":
        pairs, count, _ = binding.validate_plan(*trace, s["plan"], capacity=s["cap"], check=False,
                                                status=st, workspace=s["ws"], out=s["pairs"])
        return pairs, count, st
    if op == "probe":
        out = binding.probe_plan(*trace, s["plan"], s["num_ops"], s["slab"], check=False,
                                 out=s["out"], status=st, workspace=s["ws"])
        return out, s["arena"], st
    if op == "live_bump":
        live = binding.live_bytes_profile(*trace, s["num_ops"], check=False, out=s["live"],
                                          status=st, workspace=s["ws"])
        bump = binding.bump_plan(*trace, s["num_ops"], check=False, out=s["bump"], status=st,
                                 workspace=s["bws"])
        return live, bump, st
    if op == "breadth":
        out = binding.plan_breadth_batch(s["begin"], s["ops"], *trace, policy=s["policy"],
                                         check=False, out=s["out"], status=st)
        return out, st
    off, peak = binding.optimal_batch(s["begin"], s["ops"], *trace, check=False, out=s["out"],
                                      status=st)
    _, count, _ = binding.validate_batch(s["begin"], *trace, off, capacity=s["cap"], check=False,
                                         status=st, workspace=s["vws"], out=s["pairs"])
    return peak, count, st


def work(case):
    """Each input read once and each output written once; a slab's bytes once.
    No floating point."""
    n, k = case["n"], case["traces"]
    if case["op"] in ("batch",) and k > 1:  # lengths log-uniform over [n / 32, n]
        n = n * (31 / 32) / math.log(32)
    total = n * k
    ops = {"decode": total / 25, "ranking": total / 10}.get(case["kind"], total)
    per = {"trace": 24, "batch": 24, "step": 48, "validate": 24, "probe": 25, "live_bump": 40,
           "breadth": 24, "optimal": 40}[case["op"]]
    extra = {"batch": 28 * k, "step": 36 * k, "breadth": 20 * k, "optimal": 28 * k,
             "live_bump": 8 * ops,
             # peak of the plan: about the bytes alive at once
             "probe": {"decode": 17.0 * total, "ranking": 52e6 * min(1.0, total / 5000)}.get(
                 case["kind"], 0)}.get(case["op"], 0)
    return {"bytes": per * total + extra, "flops": 0}


def tolerance(case):
    return "exact"


def _greedy(size, first, last, best):
    """Size descending, then first op, then id; each at the lowest (or the tightest) gap."""
    n = len(size)
    off = np.zeros(n, np.int64)
    placed = np.zeros(n, bool)
    for t in sorted(range(n), key=lambda i: (-size[i], first[i], i)):
        hit = np.nonzero(placed & (first <= last[t]) & (first[t] <= last))[0]
        hit = hit[np.argsort(off[hit], kind="stable")]
        at, x, gap = 0, None, None
        for j in hit:
            room = off[j] - at
            if room >= size[t] and (x is None or (best and room < gap)):
                x, gap = at, room
                if not best:
                    break
            at = max(at, off[j] + size[j])
        off[t] = at if x is None else x
        placed[t] = True
    return off, np.int64((off + size).max() if n else 0)


def _live(size, first, last, ops):
    delta = np.zeros(ops + 1, np.int64)
    np.add.at(delta, first, size)
    np.add.at(delta, last.astype(np.int64) + 1, -size)
    return np.cumsum(delta)[:ops]


def exact(case, seed):
    """The same whole numbers from plain numpy, where that takes seconds."""
    begin, ops, size, first, last = _inputs(case, seed)
    op, status = case["op"], np.zeros(1, np.int32)
    if op == "live_bump":
        live = _live(size, first, last, int(ops.max()))
        order = np.argsort(first, kind="stable")
        off = np.zeros_like(size)
        off[order] = np.cumsum(size[order]) - size[order]
        return (live, np.array([live.max()])), (off, np.array([size.sum()])), status
    if op in ("trace", "batch") and len(size) <= 6000:
        plans, bound = [], []
        for b in range(len(ops)):
            lo, hi = begin[b], begin[b + 1]
            part = size[lo:hi], first[lo:hi], last[lo:hi]
            plans.append(_greedy(*part, case["policy"] == "best"))
            bound.append(_live(*part, int(ops[b])).max())
        out = np.concatenate([p[0] for p in plans]), np.array([p[1] for p in plans])
        return out + ((np.array(bound),) if op == "batch" else ()), status
    return None
