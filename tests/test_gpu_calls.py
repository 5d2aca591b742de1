"""Single calls read their descriptors from a few slots of pinned memory per thread: more
calls in flight than slots, on several streams and from threads that end, batches on both
sides of a slot's size, and maps between them, each against the oracle."""
import random
import sys
import threading

import pytest

import oracle
import workloads as W
from test_gpu_groups import random_forms

pytestmark = pytest.mark.gpu


def say(*a):
    print("[gpu-case]", *a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module")
def tm():
    import torch
    assert torch.cuda.is_available()
    import paper_2507_17087_amd as m
    m.lib()
    return m


def batches(n, seed):
    forms, rng = list(random_forms(60, seed, 2, 30)), random.Random(seed)
    return [W.batch(rng.sample(forms, rng.randint(1, 60))) for _ in range(n)]


def in_flight(tm, cands, streams, fail):
    import torch
    st = W.stencil((1, 2), 8)
    try:
        sts = [torch.cuda.Stream() for _ in range(streams)]
        got = []
        for i, c in enumerate(cands):
            with torch.cuda.stream(sts[i % streams]):
                if i % 5 == 4:
                    got.append((c, tm.tm_proc_map(c[0])))
                else:
                    got.append((c, tm.tm_eval_stencil_batch(c, st)))
        torch.cuda.synchronize()
        for i, (c, g) in enumerate(got):
            e = oracle.proc_map(c[0]) if i % 5 == 4 else oracle.stencil_cost_batch(c, st)
            assert (g.cpu().numpy() == e).all(), i
    except BaseException as e:  # noqa: BLE001  (reported by the test)
        fail.append(e)


@pytest.mark.parametrize("streams", [1, 3])
def test_more_calls_than_slots(tm, streams):
    say("calls in flight on", streams, "streams")
    fail = []
    in_flight(tm, batches(40, streams), streams, fail)
    assert not fail, fail


def test_threads(tm):
    say("calls from four threads, twice")
    for rep in range(2):
        fail = []
        ts = [threading.Thread(target=in_flight, args=(tm, batches(12, 10 * rep + i), 1 + i % 2, fail)) for i in range(4)]
        [t.start() for t in ts]
        [t.join() for t in ts]
        assert not fail, fail


@pytest.mark.parametrize("n", [1170, 1171, 2500])
def test_batches_around_a_slot(tm, n):
    """1,170 descriptors of 896 bytes fill a slot."""
    say("batch of", n)
    forms = list(random_forms(50, 7, 2, 30))
    cands, st = W.batch([forms[i % 50] for i in range(n)]), W.stencil((2, 1), 4)
    exp = oracle.stencil_cost_batch(W.batch(forms), st)
    got = tm.tm_eval_stencil_batch(cands, st).cpu().numpy()
    assert all((got[i::50] == exp[i]).all() for i in range(50))
    pairs = W.batch([forms[0]] * n)
    got = tm.tm_eval_redistribution_batch(pairs, pairs, 4).cpu().numpy()
    assert not got.any()
