"""The evaluation over coordinate groups, bit-exact against the oracle where its forms
meet: launch dims with several block projections (coinciding change points), block and
cyclic ones together, several cyclic sizes (their least common multiple), sizes above the
extent, blocks narrower than the halo, extents of 1; chains that are no bijections
(owners shared by several offsets); node-level counts; candidates cut into parts, whose
records exceed the launch's LDS, and batches that need two launches."""
import random
import sys

import numpy as np
import pytest

import oracle
import workloads as W
from workloads import balance_split, decompose, merge, split, swap

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


def random_forms(n, seed, k, most=40):
    """Random chains whose final dims are projected from random launch dims, either way."""
    rng, recs = random.Random(seed), []
    while len(recs) < n:
        nodes, gpus = rng.randint(1, 8), rng.choice([1, 2, 3, 4])
        shape, ops = [nodes, gpus], []
        for _ in range(rng.randint(0, 6)):
            kind = rng.choice(["split", "balance", "merge", "swap"])
            if kind in ("merge", "swap") and len(shape) > 1:
                p, q = sorted(rng.sample(range(len(shape)), 2))
                if kind == "swap":
                    shape[p], shape[q] = shape[q], shape[p]
                else:
                    shape[p] *= shape.pop(q)
                ops.append(swap(p, q) if kind == "swap" else merge(p, q))
            elif kind in ("split", "balance") and len(shape) < 7:
                i = rng.randrange(len(shape))
                s = shape[i]
                d = rng.choice([x for x in range(1, s + 1) if s % x == 0]) if kind == "split" else rng.randint(1, s + 1)
                shape[i:i + 1] = [d, -(-s // d)]
                ops.append(split(i, d) if kind == "split" else balance_split(i, d))
        ext = [rng.randint(1, most if d < 2 else 9) for d in range(k)]
        c = W.candidate(ext, nodes, gpus, ops, [(rng.randrange(k), rng.choice([W.BLOCK, W.CYCLIC])) for _ in shape])
        if oracle.validate(c)[0] == 0:
            recs.append(c)
    return W.batch(recs)


@pytest.mark.parametrize("halo", [1, 2, 3, 4])
@pytest.mark.parametrize("k", [1, 2, 3, 4])
def test_random_forms(tm, k, halo):
    say("random projections: rank", k, "halo", halo)
    cands = random_forms(150, 100 * k + halo, k)
    st = W.stencil(tuple(max(0, halo - (d & 1)) for d in range(k)), 8)
    got = tm.tm_eval_stencil_batch(cands, st).cpu().numpy()
    assert (got == oracle.stencil_cost_batch(cands, st)).all()
    got = tm.tm_eval_stencil_node_batch(cands, st).cpu().numpy()
    assert (got == oracle.stencil_node_cost_batch(cands, st)).all()


@pytest.mark.parametrize("cells_per_item", [0, 64, 1000])
@pytest.mark.parametrize("F", [(4096, 1), (1, 4096), (64, 64)])
def test_parts_and_record_ranges(tm, F, cells_per_item):
    """4,096 processors: up to 4,096 groups along one dim (records of a range at a time)
    in one workgroup or several parts; once as a bijection, once folded by a
    balance_split."""
    import torch
    say("parts", F, cells_per_item)
    ext = (5000, 9) if F[0] > F[1] else ((9, 5000) if F[1] > F[0] else (150, 130))
    cands = W.batch([W.candidate(ext, 512, 8, [merge(0, 1), decompose(0, F)]),
                     W.candidate(ext, 512, 8, [merge(0, 1), decompose(0, F), merge(0, 1), balance_split(0, 70)]),
                     W.candidate(ext, 512, 8, [merge(0, 1), decompose(0, F)], [(0, W.CYCLIC), (1, W.BLOCK)])])
    st = W.stencil((2, 1), 8)
    plan = tm.Plan(4, 1)
    plan.load(cands, st, cells_per_item=cells_per_item)
    out = torch.full((len(cands), 4), -1, dtype=torch.int64, device="cuda")
    best = torch.empty(1, dtype=torch.int64, device="cuda")
    for _ in range(2):
        plan.run(out, best)
    exp = oracle.stencil_cost_batch(cands, st)
    assert (out.cpu().numpy() == exp).all()
    assert int(best.cpu()[0]) == oracle.select_best(exp)
    plan.close()


def test_two_launches(tm):
    """A large batch with a few candidates above the one-wave launch's LDS."""
    import torch
    say("two launches")
    cands = W.random_candidates(2100, seed=77, ranks=(2, 3), octaves=(2, 4), nodes_max=16, cyclic_pct=25)
    for i, F in ((0, (64, 64)), (1049, (4096, 1)), (2099, (16, 256))):
        cands[i] = W.candidate((70, 300), 512, 8, [merge(0, 1), decompose(0, F)])
    st = W.stencil((1, 1, 1), 8)
    exp = oracle.stencil_cost_batch(cands[cands["lrank"] == 2], W.stencil((1, 1), 8))
    plan = tm.Plan(len(cands), 1)
    plan.load(cands, st)
    out = torch.empty((len(cands), 4), dtype=torch.int64, device="cuda")
    best = torch.empty(1, dtype=torch.int64, device="cuda")
    plan.run(out, best)
    got = out.cpu().numpy()
    assert (got[cands["lrank"] == 2] == exp).all()
    assert (got[cands["lrank"] == 3] == oracle.stencil_cost_batch(cands[cands["lrank"] == 3], st)).all()
    assert int(best.cpu()[0]) == oracle.select_best(got)
    plan.close()


@pytest.mark.parametrize("halo, n", [(1, 4095), (1, 4096), (2, 8191), (2, 8192), (3, 24575), (3, 24576), (4, 24576)])
def test_workgroups_by_batch(tm, halo, n):
    """Both sides of the batch sizes from which workgroups have one wave, which keep another
    number of slots in registers."""
    say("batch of", n, "halo", halo)
    wide = W.candidate((40, 30), 64, 4, [merge(0, 1), decompose(0, (16, 16))])  # a table above 128
    forms = W.batch([wide] + [c for k in (2, 3) for c in random_forms(150, 40 + halo, k, 14)])
    pick = np.random.default_rng(n).integers(0, len(forms), n)
    pick[n // 2] = 0
    st = W.stencil((halo, halo, halo), 8)
    exp = np.zeros((len(forms), 4), np.int64)
    for k in (2, 3):
        of = forms["lrank"] == k
        exp[of] = oracle.stencil_cost_batch(forms[of], W.stencil((halo,) * k, 8))
    assert (tm.tm_eval_stencil_batch(forms[pick], st).cpu().numpy() == exp[pick]).all()


def test_more_items_than_a_grid(tm):
    """4,200 candidates cut into items of one tuple, one of them into 16,000: with one-wave
    workgroups more than 2^32 threads, so workgroups take several items."""
    import torch
    say("more items than a grid holds")
    forms = random_forms(60, 9, 2, 20)
    cands = forms[np.arange(4200) % len(forms)]
    cands[4100] = W.candidate((20000, 3), 2000, 8, [merge(0, 1), decompose(0, (16000, 1))])
    st = W.stencil((1, 1), 8)
    exp = oracle.stencil_cost_batch(forms, st)[np.arange(4200) % len(forms)]
    exp[4100] = oracle.stencil_cost_batch(cands[4100:4101], st)[0]
    plan = tm.Plan(len(cands), 1)
    plan.load(cands, st, cells_per_item=1)
    assert plan.info()[1] > 16000
    out = torch.full((len(cands), 4), -1, dtype=torch.int64, device="cuda")
    best = torch.empty(1, dtype=torch.int64, device="cuda")
    plan.run(out, best)
    assert (out.cpu().numpy() == exp).all()
    assert int(best.cpu()[0]) == oracle.select_best(exp)
    plan.close()
