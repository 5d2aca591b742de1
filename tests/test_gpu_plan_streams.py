"""A plan used on several streams at once: what is in flight on one does not change what
another gets."""
import sys

import numpy as np
import pytest

import oracle
import workloads as W

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


def menu(extent=(96, 200, 130)):
    return W.c2_candidates(oracle.enumerate_factorizations(128, 3), extent=extent)


def loaded(tm, cands, st):
    import torch
    plan = tm.Plan(len(cands), 1)
    plan.load(cands, st)
    out = torch.empty((len(cands), 4), dtype=torch.int64, device="cuda")
    best = torch.empty(1, dtype=torch.int64, device="cuda")
    return plan, out, best


def test_maps_in_flight(tm):
    """Maps of different candidates of one plan, one after another on each of three streams."""
    import torch
    say("maps in flight")
    cands, n = menu()[::7], 96 * 200 * 130
    plan, out, best = loaded(tm, cands, W.stencil((1, 1, 1), 8))
    plan.run(out, best)
    ref = [torch.from_numpy(oracle.proc_map(c).ravel()) for c in cands]
    sts = [torch.cuda.Stream() for _ in range(3)]
    maps = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in cands]
    idx = torch.arange(len(cands), dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    for i, m in enumerate(maps):
        with torch.cuda.stream(sts[i % 3]):
            plan.materialize(m, **({"d_index": idx[i:i + 1]} if i % 2 else {"index": i}))
    torch.cuda.synchronize()
    assert all(torch.equal(m.cpu(), r) for m, r in zip(maps, ref))
    plan.close()


def test_run_map_beside_maps(tm):
    """Runs with the winner's map on one stream, maps of other candidates on another."""
    import torch
    say("run and map beside other maps")
    cands, n, st = menu()[::5], 96 * 200 * 130, W.stencil((1, 2, 1), 8)
    plan, out, best = loaded(tm, cands, st)
    exp = oracle.stencil_cost_batch(cands, st)
    win = oracle.select_best(exp)
    others = [i for i in range(len(cands)) if i != win][:8]
    maps = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in others]
    wmap = torch.empty(n, dtype=torch.int32, device="cuda")
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(a):
        plan.run_map(out, best, wmap)
    torch.cuda.synchronize()
    for i, m in zip(others, maps):
        with torch.cuda.stream(a):
            plan.run_map(out, best, wmap)
        with torch.cuda.stream(b):
            plan.materialize(m, index=i)
    torch.cuda.synchronize()
    assert (out.cpu().numpy() == exp).all() and int(best.cpu()[0]) == win
    assert (wmap.cpu().numpy() == oracle.proc_map(cands[win]).ravel()).all()
    assert all((m.cpu().numpy() == oracle.proc_map(cands[i]).ravel()).all() for i, m in zip(others, maps))
    plan.close()


@pytest.mark.parametrize("n", [5, 64, 96])
def test_runs_in_flight(tm, n):
    """Runs of one plan on three streams at once, with outputs of their own, several rounds
    and then one alone: each counts its own finished workgroups."""
    import torch
    say("runs in flight", n)
    forms, st = menu((40, 70, 33)), W.stencil((2, 1, 2), 8)
    cands = forms[(np.arange(n) * 11 + 3) % len(forms)]
    plan, out, best = loaded(tm, cands, st)
    exp = oracle.stencil_cost_batch(cands, st)
    win = oracle.select_best(exp)
    sts = [torch.cuda.Stream() for _ in range(3)]
    for rnd in range(4):
        outs = [torch.zeros_like(out) for _ in range(45)]
        wins = [torch.full_like(best, -9) for _ in outs]
        torch.cuda.synchronize()
        for i, (o, w) in enumerate(zip(outs, wins)):
            with torch.cuda.stream(sts[i % 3]):
                plan.run(o, w)
        torch.cuda.synchronize()
        assert all((o.cpu().numpy() == exp).all() for o in outs), rnd
        assert [int(w.cpu()[0]) for w in wins] == [win] * len(wins), rnd
        plan.run(out.zero_(), best.fill_(-9))
        assert (out.cpu().numpy() == exp).all() and int(best.cpu()[0]) == win
    plan.close()
