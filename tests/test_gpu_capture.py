"""What a caller's graph can record: a loaded plan's calls, whose replays equal the eager
results; single calls, whose descriptors do not outlive the call, are refused and leave the
capture whole."""
import contextlib
import gc
import sys
import threading

import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_volumes import huge

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


@contextlib.contextmanager
def recording():
    """A graph being captured.  Nothing is garbage-collected meanwhile: a graph or a plan of
    an earlier test would be destroyed, which waits for the device (and so would be the last
    graph of a loop, when the next one takes its name)."""
    import torch
    g = torch.cuda.CUDAGraph()
    gc.collect()
    gc.disable()
    try:
        with torch.cuda.graph(g):
            yield g
    finally:
        gc.enable()


def code_of(tm, call):
    """The error code of a call, 0 if it succeeds; no reference to its frames is kept."""
    try:
        call()
    except tm.TaskmapError as e:
        return e.code
    return 0


def batch():
    cands = W.c2_candidates(oracle.enumerate_factorizations(128, 3), extent=(24, 40, 17))[3:150:9]
    st = W.stencil((1, 2, 1), 8)
    return cands, st, oracle.stencil_cost_batch(cands, st)


@pytest.mark.parametrize("before", [False, True])
def test_single_calls_are_refused(tm, before):
    """before: the thread has its staging memory and slots already."""
    import torch
    say("single calls under capture", before)
    cands, st, exp = batch()
    big = W.batch([cands[0], W.candidate((24, 40, 17), 16, 8, [W.merge(0, 1), W.balance_split(0, 33000)])])
    many = cands[[i % len(cands) for i in range(1200)]]
    costs = torch.from_numpy(exp).cuda()
    rows = torch.zeros((len(many), 4), dtype=torch.int64, device="cuda")
    calls = [lambda: tm.tm_eval_stencil_batch(cands, st, rows), lambda: tm.tm_eval_stencil_batch_noalloc(cands, st, rows),
             lambda: tm.tm_eval_stencil_batch(many, st, rows),
             lambda: tm.tm_eval_stencil_node_batch(cands, st, rows), lambda: tm.tm_proc_map(cands[0]),
             lambda: tm.tm_chain_table(cands[0]), lambda: tm.tm_eval_matmul_batch(cands, 8),
             lambda: tm.tm_eval_matmul_batch(W.batch([huge((6, 5, 4), 2, 2)]), 8),
             lambda: tm.tm_eval_redistribution_batch(cands, cands, 8, rows),
             lambda: tm.tm_eval_redistribution_batch(big, big, 8, rows),
             lambda: tm.tm_select_best(costs, [0, 3, len(cands)])]
    if before:
        for c in calls:
            c()
    plan = tm.Plan(len(cands), 1)
    plan.load(cands, st)
    out = torch.zeros((len(cands), 4), dtype=torch.int64, device="cuda")
    best = torch.zeros(1, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    codes = []
    with recording() as g:
        codes += [code_of(tm, c) for c in calls]
        plan.run(out, best)
    assert codes == [tm.TM_ENOTSUP] * len(calls)
    for _ in range(3):
        assert (tm.tm_eval_stencil_batch(cands, st, out.zero_()).cpu().numpy() == exp).all()
        out.zero_(), best.fill_(-3)
        g.replay()
        torch.cuda.synchronize()
        assert (out.cpu().numpy() == exp).all() and int(best.cpu()[0]) == oracle.select_best(exp)
    plan.close()


@pytest.mark.parametrize("calls", ["map", "map-at-index", "run-map", "all"])
@pytest.mark.parametrize("reload", [False, True])
def test_maps_after_a_run(tm, calls, reload):
    """The first maps of a plan, recorded after a run of it: reload, of a larger batch after
    the smaller one's map."""
    import torch
    say("captured", calls, "after a reload" if reload else "")
    cands, st, exp = batch()
    n, win = 24 * 40 * 17, oracle.select_best(exp)
    other = (win + 2) % len(cands)
    plan = tm.Plan(len(cands), 1)
    out = torch.zeros((len(cands), 4), dtype=torch.int64, device="cuda")
    best = torch.zeros(1, dtype=torch.int64, device="cuda")
    wmap, omap, smap = (torch.zeros(n, dtype=torch.int32, device="cuda") for _ in range(3))
    if reload:
        plan.load(cands[:2], st)
        plan.run(out, best)
        plan.materialize(smap, index=1)
    plan.load(cands, st)
    plan.run(out, best)
    torch.cuda.synchronize()
    with recording() as g:
        if calls == "run-map":
            plan.run_map(out, best, wmap)
        elif calls == "all":
            plan.run(out, best)
        if calls in ("map", "all"):
            plan.materialize(wmap, d_index=best)
        if calls in ("map-at-index", "all"):
            plan.materialize(omap, index=other)
    for _ in range(4):
        wmap.fill_(-1), omap.fill_(-1)
        if calls in ("run-map", "all"):
            out.zero_(), best.fill_(-1)
        plan.materialize(smap, index=(other + 1) % len(cands))  # the plan's own work in between
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert (out.cpu().numpy() == exp).all() and int(best.cpu()[0]) == win
        if calls != "map-at-index":
            assert (wmap.cpu().numpy() == oracle.proc_map(cands[win]).ravel()).all()
        if calls in ("map-at-index", "all"):
            assert (omap.cpu().numpy() == oracle.proc_map(cands[other]).ravel()).all()
    if reload:
        assert (smap.cpu().numpy() == oracle.proc_map(cands[(other + 1) % len(cands)]).ravel()).all()
    plan.close()


@pytest.mark.parametrize("n", [700, 5000])
@pytest.mark.parametrize("first", ["forward", "grad"])
def test_ranker_after_the_other_call(tm, first, n):
    """A forward pass recorded where only gradients were taken before, and the other way
    round; rows in the range of the buffers' smallest size and beyond."""
    import torch
    say("captured ranker call after", first, n)
    gen = torch.Generator().manual_seed(5)
    rk, ref = tm.Ranker(seed=4), tm.Ranker(seed=4)
    feat, target = torch.randn((n, 64), generator=gen).cuda(), torch.randn((n, 2), generator=gen).cuda()
    calls = [lambda r: r.forward(feat), lambda r: r.grad(feat, target)]
    if first == "grad":
        calls.reverse()
    exp = calls[1](ref)
    calls[0](rk)
    torch.cuda.synchronize()
    with recording() as g:
        got = calls[1](rk)
    for _ in range(3):
        got.fill_(7)
        calls[0](rk)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, exp)
    rk.close(), ref.close()


@pytest.mark.parametrize("warm", [True, False])
def test_thread_ends_during_a_capture(tm, warm):
    """Another thread's single calls, and the end of that thread, while this one captures;
    warm: it has made calls before."""
    import torch
    say("a thread ends during a capture", warm)
    cands, st, exp = batch()
    plan = tm.Plan(len(cands), 1)
    plan.load(cands, st)
    out, theirs = (torch.zeros((len(cands), 4), dtype=torch.int64, device="cuda") for _ in range(2))
    best = torch.zeros(1, dtype=torch.int64, device="cuda")
    many = cands[[i % len(cands) for i in range(1200)]]
    rows = torch.zeros((1200, 4), dtype=torch.int64, device="cuda")
    pmap = torch.zeros(24 * 40 * 17, dtype=torch.int32, device="cuda")
    side, ready, go, fail = torch.cuda.Stream(), threading.Event(), threading.Event(), []

    def calls():
        with torch.cuda.stream(side):
            for _ in range(6):
                tm.tm_eval_stencil_batch(cands, st, theirs)
                tm.tm_proc_map(cands[4], pmap)
                tm.tm_eval_stencil_batch(many, st, rows)  # larger than a slot

    def work():
        try:
            if warm:
                calls()
                side.synchronize()
            ready.set()
            go.wait(60)
            calls()
        except BaseException as e:  # noqa: BLE001  (reported by the test)
            fail.append(repr(e))
            ready.set()

    th = threading.Thread(target=work)
    th.start()
    assert ready.wait(60) and not fail, fail
    torch.cuda.synchronize()
    with recording() as g:
        plan.run(out, best)
        go.set()
        th.join()
        plan.materialize(pmap, d_index=best)
    assert not fail, fail
    torch.cuda.synchronize()
    assert (theirs.cpu().numpy() == exp).all()
    assert (rows.cpu().numpy() == exp[np.arange(1200) % len(exp)]).all()
    assert (pmap.cpu().numpy() == oracle.proc_map(cands[4]).ravel()).all()
    g.replay()
    torch.cuda.synchronize()
    win = oracle.select_best(exp)
    assert (out.cpu().numpy() == exp).all() and int(best.cpu()[0]) == win
    assert (pmap.cpu().numpy() == oracle.proc_map(cands[win]).ravel()).all()
    plan.close()
