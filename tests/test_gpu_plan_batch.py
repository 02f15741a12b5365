"""Parity of the batched HIP planner (mp_plan_batch) with the CPU oracle.

Integer work: offsets, peaks and lower bounds must match bit for bit."""
import numpy as np
import pytest

import oracle
from gpu_util import batch_to_device, dev, host, need_gpu, torch
from paper_2203_00448_amd import tracegen as tg

pytestmark = pytest.mark.gpu


def _oracle_batch(batch):
    off, peak = oracle.plan_batch(batch.begin, batch.num_ops, batch.size, batch.first, batch.last)
    lb = np.array([oracle.live_bytes_profile(*[a for a in (batch.trace(b).size, batch.trace(b).first,
                                                            batch.trace(b).last)],
                                             batch.trace(b).num_ops)[1]
                   for b in range(batch.n_traces)], dtype=np.int64)
    return off, peak, lb


def _gpu_batch(binding, batch, **kw):
    args = batch_to_device(batch)
    off, peak, lb = binding.plan_batch(*args, **kw)
    return host(off), host(peak), host(lb)


def _check(binding, batch, **kw):
    off, peak, lb = _gpu_batch(binding, batch, **kw)
    eo, ep, el = _oracle_batch(batch)
    bad = np.nonzero(off != eo)[0]
    assert bad.size == 0, f"{bad.size} offsets differ, first at {bad[:5]}"
    assert (peak == ep).all()
    assert (lb == el).all()
    return off, peak, lb


def test_chain256_single_trace_batch():
    binding = need_gpu()
    print("case chain256 as a batch of one", flush=True)
    _check(binding, tg.concat([tg.chain256()]))


def test_resnext_batch_full():
    binding = need_gpu()
    print("case resnext batch 1024 x 2000", flush=True)
    batch = tg.resnext_batch()
    off, peak, lb = _check(binding, batch, max_trace_len=2000)
    assert (peak >= lb).all()


def test_random_ragged_batches():
    binding = need_gpu()
    rng = np.random.default_rng(100)
    traces = []
    for k in range(300):
        n = int(rng.choice([0, 1, 2, 3, 17, 64, 255, 256, 257, 700, 1500]))
        if n <= 64:   # dense: up to n^2/2 pairs
            T, span = int(rng.integers(1, 20)), int(rng.integers(1, 20))
        else:         # about one birth per op, short lifetimes
            T, span = n * int(rng.integers(1, 3)) + 1, int(rng.integers(1, 12))
        alphabet = [64, 128, 192, 448, 1024] if k % 3 == 0 else None
        traces.append(tg.random_trace(rng, n, T, max_len=span, sizes=alphabet,
                                      sorted_first=(k % 2 == 0)))
    print("case 300 random ragged traces (sorted and unsorted first)", flush=True)
    _check(binding, tg.concat(traces), max_trace_len=1500)


def test_adversarial_shapes():
    binding = need_gpu()
    rng = np.random.default_rng(101)
    n = 200
    full = tg.Trace(64 * rng.integers(1, 50, n), np.zeros(n, np.int32), np.full(n, 9, np.int32), 10)
    equal = tg.random_trace(rng, 600, 300, max_len=10, sizes=[320])
    disjoint = tg.Trace(64 * rng.integers(1, 50, n), np.arange(n, dtype=np.int32),
                        np.arange(n, dtype=np.int32), n)
    span = tg.random_trace(rng, 500, 100, max_len=5, sorted_first=True)
    span.first[250], span.last[250] = 0, 99
    odd = tg.random_trace(rng, 300, 50, max_len=10, sizes=[1, 3, 7, 100, 1001])
    print("case adversarial shapes", flush=True)
    _check(binding, tg.concat([full, equal, disjoint, span, odd]), max_trace_len=1000)


def test_max_trace_len_4096():
    binding = need_gpu()
    rng = np.random.default_rng(102)
    t = tg.random_trace(rng, 4096, 4096, max_len=4, sorted_first=True)
    print("case 4096-tensor trace", flush=True)
    _check(binding, tg.concat([t, tg.resnext_trace(5)]), max_trace_len=4096)


def test_deterministic_repeats():
    binding = need_gpu()
    batch = tg.concat(tg.resnext_trace(b) for b in range(64))
    args = batch_to_device(batch)
    print("case 10 repeats of 64 resnext traces", flush=True)
    ref = [host(x) for x in binding.plan_batch(*args, max_trace_len=2000)]
    for _ in range(10):
        got = [host(x) for x in binding.plan_batch(*args, max_trace_len=2000)]
        for a, b in zip(ref, got):
            assert np.array_equal(a, b)


def _status(binding, batch, **kw):
    args = batch_to_device(batch)
    status = binding.new_status()
    binding.plan_batch(*args, check=False, status=status, **kw)
    return int(status.item())


def test_device_status_codes():
    binding = need_gpu()
    good = tg.chain256()
    print("case device status codes", flush=True)
    assert _status(binding, tg.concat([good])) == binding.MP_OK
    bad = tg.Trace(good.size.copy(), good.first.copy(), good.last.copy(), good.num_ops)
    bad.size[7] = 0
    assert _status(binding, tg.concat([good, bad])) == binding.MP_EINVAL
    bad = tg.Trace(good.size.copy(), good.first.copy(), good.last.copy(), good.num_ops)
    bad.first[3] = bad.last[3] + 1
    assert _status(binding, tg.concat([bad])) == binding.MP_EINVAL
    bad = tg.Trace(good.size.copy(), good.first.copy(), good.last.copy(), 200)
    assert _status(binding, tg.concat([bad])) == binding.MP_EINVAL  # last >= num_ops
    big = tg.Trace(np.array([2 ** 62, 2 ** 62], np.int64), np.zeros(2, np.int32),
                   np.zeros(2, np.int32), 1)
    assert _status(binding, tg.concat([good, big])) == binding.MP_EOVERFLOW
    # more tensors than the declared maximum trace length
    assert _status(binding, tg.concat([good]), max_trace_len=100) == binding.MP_EINVAL
    # sizes past 32-bit unit counts and more pairs than the LDS lists hold are
    # planned, not refused (general path; parity in test_gpu_batch_general.py)
    wide = tg.Trace(np.array([2 ** 31 + 1, 2 ** 31 + 1], np.int64), np.zeros(2, np.int32),
                    np.zeros(2, np.int32), 1)
    n = 2000
    dense = tg.Trace(np.full(n, 64, np.int64), np.zeros(n, np.int32), np.zeros(n, np.int32), 1)
    assert _status(binding, tg.concat([wide, dense])) == binding.MP_OK


def test_empty_batch_and_empty_traces():
    binding = need_gpu()
    batch = tg.concat([tg.Trace(np.zeros(0, np.int64), np.zeros(0, np.int32), np.zeros(0, np.int32), 0)] * 3)
    off, peak, lb = _gpu_batch(binding, batch, max_trace_len=0)
    assert off.shape == (0,) and peak.tolist() == [0, 0, 0] and lb.tolist() == [0, 0, 0]
    batch = tg.concat([])
    off, peak, lb = _gpu_batch(binding, batch, max_trace_len=0)
    assert off.shape == (0,) and peak.shape == (0,)


def test_one_slot_unsorted_full_bound():
    """An unsorted 255-tensor trace with 85 ops and lifetimes of up to 8 ops,
    alone in a batch whose bound is its own length (one slot a thread).  With an
    odd bound the predecessor counts -- LDS words that atomics add to -- once
    started halfway through a word; this case had ended in a memory aperture
    violation."""
    binding = need_gpu()
    rng = np.random.default_rng(300)
    t = tg.random_trace(rng, 255, 85, max_len=8, sizes=[64, 192, 448])
    _check(binding, tg.concat([t]), max_trace_len=255)


@pytest.mark.parametrize("bound", [3, 31, 257, 1023, 2047, 4095])
def test_odd_bounds(bound):
    """Odd bounds (the default bound is the longest trace's length): a trace of
    the bound's length, recorded and in any order, under both fits."""
    binding = need_gpu()
    rng = np.random.default_rng(304)
    traces = [tg.random_trace(rng, bound, bound, max_len=6, sorted_first=s, sizes=[64, 192, 448])
              for s in (True, False)]
    batch = tg.concat(traces)
    for policy in (oracle.LOWEST_FIT, oracle.BEST_FIT):
        print(f"case odd bound {bound}, policy {policy}", flush=True)
        off, peak, _ = binding.plan_batch(*batch_to_device(batch), policy=policy)
        eo, ep = oracle.plan_batch(batch.begin, batch.num_ops, batch.size, batch.first,
                                   batch.last, policy)
        assert np.array_equal(host(off), eo) and np.array_equal(host(peak), ep)


@pytest.mark.parametrize("call", ["lowest", "best", "breadth", "dense"])
def test_refused_begin_with_shared_tensors(call):
    """A begin[] that goes back gives several traces the same tensors.  The call
    is refused, and until then each of those traces keeps to its own memory: its
    working data lies in no array that another one of them writes, so the ids it
    reads are ids of its tensors and the plan (the same for all of them, in any
    order) is the oracle's.  "dense" takes the general path, whose lists the
    traces share: there the call only has to end in MP_EINVAL."""
    binding = need_gpu()
    rng = np.random.default_rng(170)
    n, copies = 1500, 300
    if call == "dense":
        t = tg.random_trace(rng, n, 40, max_len=30)
    else:
        t = tg.random_trace(rng, n, n, max_len=6)  # in any order
    assert np.any(np.diff(t.first) < 0)
    begin = np.array(([0, n] * copies)[: 2 * copies], np.int64)
    ops = np.full(begin.size - 1, t.num_ops, np.int32)
    args = (dev(begin, torch.int64), dev(ops, torch.int32), dev(t.size, torch.int64),
            dev(t.first, torch.int32), dev(t.last, torch.int32))
    st = binding.new_status()
    peak = torch.full((ops.size,), -7, dtype=torch.int64, device="cuda")
    off = torch.full((n,), -7, dtype=torch.int64, device="cuda")
    print(f"case refused begin, {call}", flush=True)
    if call == "breadth":
        binding.plan_breadth_batch(*args, check=False, status=st, out=(off, peak))
        eo, ep = oracle.plan_breadth(t.size, t.first, t.last, t.num_ops, 0)
    else:
        policy = int(call == "best")
        binding.plan_batch(*args, max_trace_len=n, policy=policy, check=False, status=st,
                           out=(off, peak, None))
        eo, ep = oracle.plan_trace(t.size, t.first, t.last, t.num_ops, policy)
    assert int(st.item()) == binding.MP_EINVAL
    if call != "dense":
        assert np.array_equal(host(off), eo)
        assert np.all(host(peak)[::2] == ep) and np.all(host(peak)[1::2] == -7)
