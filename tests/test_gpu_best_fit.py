"""Parity of the BEST_FIT policy on the GPU with the CPU oracle.

BEST_FIT is the tightest-gap reading of the best-fit rule of
Section 2.3: among the free gaps left by the already placed, lifetime-
intersecting tensors, the smallest one that holds the tensor (lowest start
among equals), the space above all of them only when no gap holds it.
Integer work: offsets and peaks must match the oracle bit for bit.  The
batched planner fits a tensor with up to 256 lifetime-intersecting tensors in
one wave and plans a trace with a larger one on its general path."""
import hashlib
import json
import os

import numpy as np
import pytest

import oracle
from gpu_util import batch_to_device, dev, host, need_gpu, torch
from paper_2203_00448_amd import tracegen as tg

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))
BEST = oracle.BEST_FIT


def _sha(a):
    return hashlib.sha256(np.ascontiguousarray(a).astype("<i8").tobytes()).hexdigest()


def _check_batch(binding, batch, **kw):
    args = batch_to_device(batch)
    off, peak, lb = binding.plan_batch(*args, policy=binding.BEST_FIT, **kw)
    off, peak = host(off), host(peak)
    eo, ep = oracle.plan_batch(batch.begin, batch.num_ops, batch.size, batch.first, batch.last,
                               BEST)
    bad = np.nonzero(off != eo)[0]
    assert bad.size == 0, f"{bad.size} offsets differ, first at {bad[:5]}"
    assert np.array_equal(peak, ep)
    return off, peak


def _hand_traces():
    with open(os.path.join(HERE, "golden", "hand_examples.json")) as fh:
        ex = json.load(fh)["examples"]
    out = []
    for e in ex:
        f = np.asarray(e["first"], np.int32)
        out.append((e, tg.Trace(np.asarray(e["size"], np.int64), f,
                                np.asarray(e["last"], np.int32), int(max(e["last"])) + 1)))
    return out


def test_hand_examples_batch_and_trace():
    binding = need_gpu()
    print("case hand examples, BEST_FIT", flush=True)
    hand = _hand_traces()
    off, _ = _check_batch(binding, tg.concat([t for _, t in hand]), max_trace_len=16)
    batch = tg.concat([t for _, t in hand])
    for k, (e, t) in enumerate(hand):
        lo, hi = int(batch.begin[k]), int(batch.begin[k + 1])
        assert off[lo:hi].tolist() == e["best_fit"], e["name"]
        o, p = binding.plan_trace(dev(t.size, torch.int64), dev(t.first, torch.int32),
                                  dev(t.last, torch.int32), t.num_ops, policy=binding.BEST_FIT)
        assert host(o).tolist() == e["best_fit"], e["name"]
    # the policies differ on E4: id 4 takes the tight gap [256, 320)
    e4 = [e for e, _ in hand if e["name"] == "E4"][0]
    assert e4["best_fit"] != e4["lowest_fit"]


def test_chain256_against_stored_digest():
    binding = need_gpu()
    print("case chain256, BEST_FIT", flush=True)
    with open(os.path.join(HERE, "golden", "expected.json")) as fh:
        exp = json.load(fh)["configs"]["chain256_best_fit"]
    t = tg.chain256()
    off, peak = _check_batch(binding, tg.concat([t]))
    assert _sha(off) == exp["offsets_sha256"] and int(peak[0]) == exp["peak"]
    o, p = binding.plan_trace(dev(t.size, torch.int64), dev(t.first, torch.int32),
                              dev(t.last, torch.int32), t.num_ops, policy=binding.BEST_FIT)
    assert _sha(host(o)) == exp["offsets_sha256"] and int(p.item()) == exp["peak"]


def test_random_ragged_batches():
    binding = need_gpu()
    rng = np.random.default_rng(400)
    traces = []
    for k in range(200):
        n = int(rng.choice([0, 1, 2, 3, 17, 64, 150, 255, 256, 257, 700, 1500]))
        if n <= 150:  # dense: up to 149 neighbours per tensor
            T, span = int(rng.integers(1, 20)), int(rng.integers(1, 20))
        else:         # about one birth per op, short lifetimes
            T, span = n * int(rng.integers(1, 3)) + 1, int(rng.integers(1, 12))
        alphabet = [64, 128, 192, 448, 1024] if k % 3 == 0 else None
        traces.append(tg.random_trace(rng, n, T, max_len=span, sizes=alphabet,
                                      sorted_first=(k % 2 == 0)))
    print("case 200 random ragged traces, BEST_FIT", flush=True)
    _check_batch(binding, tg.concat(traces), max_trace_len=1500)


def test_resnext_batch():
    binding = need_gpu()
    print("case resnext batch 1024 x 2000, BEST_FIT", flush=True)
    _check_batch(binding, tg.resnext_batch(), max_trace_len=2000)


def test_batch_neighbour_limit():
    binding = need_gpu()
    print("case one tensor meeting 299 others, BEST_FIT", flush=True)
    n = 300  # tensor 0 lives through every op, tensor i > 0 only at op i: 299 pairs
    t = tg.Trace(np.full(n, 64, np.int64), np.arange(n, dtype=np.int32),
                 np.arange(n, dtype=np.int32), n)
    t.first[0], t.last[0] = 0, n - 1
    _, peak = _check_batch(binding, tg.concat([t, tg.chain256()]))
    assert int(peak[0]) == 128


@pytest.mark.parametrize("seed", [401, 402])
def test_single_trace_random(seed):
    binding = need_gpu()
    rng = np.random.default_rng(seed)
    print(f"case single-trace random, BEST_FIT, seed {seed}", flush=True)
    for k in range(12):
        n = int(rng.choice([1, 2, 40, 700, 5000]))
        T = int(rng.integers(1, 2000))
        alphabet = [64, 128, 192, 448, 4096] if k % 3 == 0 else None
        t = tg.random_trace(rng, n, T, max_len=int(rng.integers(1, T + 1)), sizes=alphabet,
                            sorted_first=(k % 2 == 0))
        o, p = binding.plan_trace(dev(t.size, torch.int64), dev(t.first, torch.int32),
                                  dev(t.last, torch.int32), t.num_ops, policy=binding.BEST_FIT)
        eo, ep = oracle.plan_trace(t.size, t.first, t.last, t.num_ops, BEST)
        assert np.array_equal(host(o), eo) and int(p.item()) == ep


def test_decode100k_single_trace():
    binding = need_gpu()
    print("case decode100k, BEST_FIT (oracle about 10 s)", flush=True)
    t = tg.decode100k()
    o, p = binding.plan_trace(dev(t.size, torch.int64), dev(t.first, torch.int32),
                              dev(t.last, torch.int32), t.num_ops, policy=binding.BEST_FIT)
    eo, ep = oracle.plan_trace(t.size, t.first, t.last, t.num_ops, BEST)
    bad = np.nonzero(host(o) != eo)[0]
    assert bad.size == 0, f"{bad.size} offsets differ, first at {bad[:5]}"
    assert int(p.item()) == ep


def _wide_neighbourhood(K, rng, shuffle):
    """A smallest tensor t that meets K others, in whose offsets there are gaps: short
    ones, four an op, below a floor; above it six that t meets, with gaps where
    tensors that live only after t lie between them, from wide to narrow in address
    order, and the two narrowest that hold t equal."""
    T = -(-(K - 6) // 4)
    first, last, size = [0], [T - 1], [50]                    # t
    for i in range(K - 6):
        first.append(i // 4), last.append(i // 4), size.append(int(rng.integers(1300, 5000)))
    first.append(T), last.append(T + 1), size.append(20_000)  # the floor
    for met, above in ((1000, (900,)), (800, (600,)), (500, (300, 300)), (250, (120,)),
                       (110, (60, 60)), (55, ())):
        first.append(int(rng.integers(T // 4, T)))  # (so that none meets more than K)
        last.append(T + 1), size.append(met)
        for b in above:
            first.append(T), last.append(T + 1), size.append(b)
    first, last = np.array(first, np.int32), np.array(last, np.int32)
    n = first.size
    meets = ((first[:, None] <= last) & (last[:, None] >= first)).sum(axis=1) - 1
    assert meets[0] == K and meets.max() <= max(K, 48)
    p = rng.permutation(n) if shuffle else np.argsort(first, kind="stable")
    return tg.Trace(64 * np.array(size, np.int64)[p], first[p], last[p], T + 2)


@pytest.mark.parametrize("K", [7, 8, 9, 15, 16, 17, 31, 32, 63, 64, 65, 255, 256])
def test_batch_neighbour_counts(K):
    """Traces whose tensors meet K others (and, at the ends, fewer), around the
    counts at which the batched planner changes the lanes a tensor is fitted
    by; sizes of few values (equal gaps and equal ends) and of many, in order
    and shuffled; and one tensor whose K neighbours leave gaps to choose from, so
    that the two fits differ."""
    binding = need_gpu()
    rng = np.random.default_rng(700 + K)
    traces, chosen = [], []
    for sizes in ([64, 128, 192, 320], None):
        for shuffle in (False, True):
            n = 2 * K + 40
            first = np.arange(n, dtype=np.int32)
            left = K // 2  # a constant lifetime: K // 2 or so before, the rest after
            last = np.minimum(first + left + (first % 2) * (K % 2), n - 1).astype(np.int32)
            size = (np.asarray(sizes, np.int64)[rng.integers(0, 4, n)] if sizes
                    else 64 * rng.integers(1, 400, n))
            chosen += [_wide_neighbourhood(K, rng, shuffle) for _ in range(2)]
            if K > 32:  # more pairs than the lists hold
                continue
            p = rng.permutation(n) if shuffle else np.arange(n)
            traces.append(tg.Trace(size[p], first[p], last[p], n))
    for t in chosen:
        lowest, best = (oracle.plan_trace(t.size, t.first, t.last, t.num_ops, policy)[0]
                        for policy in (0, BEST))
        assert not np.array_equal(lowest, best)
    print(f"case BEST_FIT, {K} neighbours", flush=True)
    _check_batch(binding, tg.concat(traces + chosen), max_trace_len=600)
