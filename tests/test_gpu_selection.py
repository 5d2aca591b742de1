"""The winner of a batch and its map, on both sides of the sizes at which the selection moves
to a launch of its own and at which that launch's threads take more rows; every candidate
occurs several times (the first index wins), the rows lie at an address of 8 bytes only."""
import sys

import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tm():
    import torch
    assert torch.cuda.is_available()
    import paper_2507_17087_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("n", [2, 96, 97, 1024, 1025, 4096, 4097, 9000])
def test_winner_and_map(tm, n):
    import torch
    print("[gpu-case] selection over", n, "rows", file=sys.stderr, flush=True)
    menu = W.c2_candidates(oracle.enumerate_factorizations(128, 3), extent=(24, 40, 16))
    pick = np.random.default_rng(n).integers(0, len(menu), n)
    cands = menu[pick]
    st = W.stencil((1, 2, 1), 4)
    plan = tm.Plan(n, 1)
    plan.load(cands, st)
    out = torch.empty(4 * n + 1, dtype=torch.int64, device="cuda")[1:].view(n, 4)
    best = torch.empty(1, dtype=torch.int64, device="cuda")
    pmap = torch.empty(24 * 40 * 16, dtype=torch.int32, device="cuda")
    exp = oracle.stencil_cost_batch(menu, st)[pick]
    win = oracle.select_best(exp)
    for _ in range(2):
        best.fill_(-7)
        plan.run_map(out, best, pmap)
        assert (out.cpu().numpy() == exp).all()
        assert int(best.cpu()[0]) == win
        assert (pmap.cpu().numpy() == oracle.proc_map(cands[win]).ravel()).all()
    plan.close()
