"""Matmul tile fetches and redistribution volumes over coordinate groups, bit-exact
against the oracle and against the general kernels (which take a batch that holds one
mapping too large for a workgroup's LDS): random chains with several block and cyclic
projections of a dim, in either direction, bijective and not; coordinates that share a
final coordinate; pairs cut into parts; joint dims with more block sizes than a pair
lists."""
import random
import sys

import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_groups import random_forms
from workloads import balance_split, decompose, merge, split

pytestmark = pytest.mark.gpu
B, C = W.BLOCK, W.CYCLIC


def say(*a):
    print("[gpu-case]", *a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module")
def tm():
    import torch
    assert torch.cuda.is_available()
    import paper_2507_17087_amd as m
    m.lib()
    return m


def huge(ext, nodes, gpus):
    """An owner table above the LDS budget: blocks of one dim padded to 33,000."""
    return W.candidate(ext, nodes, gpus, [merge(0, 1), balance_split(0, 33000)], [(0, B), (len(ext) - 1, B)])


def matmul_rows(tm, cands, tile_bytes=3):
    pp, out = tm.tm_eval_matmul_batch(cands, tile_bytes)
    return pp.cpu().numpy(), out.cpu().numpy()


def check_matmul(tm, recs, tile_bytes=3):
    pp, out = matmul_rows(tm, W.batch(recs), tile_bytes)
    off = 0
    for i, c in enumerate(recs):
        per, tot = oracle.matmul_cost(c, tile_bytes)
        P = int(c["nodes"]) * int(c["gpus"])
        assert (pp[off:off + P] == np.asarray(per)).all(), i
        assert (out[i] == np.asarray(tot)).all(), i
        off += P
    # the general kernels' rows of the same candidates
    pg, og = matmul_rows(tm, W.batch(recs + [huge((6, 5, 4), 2, 2)]), tile_bytes)
    assert (pg[:off] == pp).all() and (og[:-1] == out).all()


def pairs_of(recs, seed):
    """Every candidate of each (domain, machine) with another one of it."""
    rng, by = random.Random(seed), {}
    for c in recs:
        by.setdefault((tuple(c["extent"]), int(c["nodes"]), int(c["gpus"])), []).append(c)
    out = []
    for same in by.values():
        other = same[:]
        rng.shuffle(other)
        out += zip(same, other)
    return out


def check_pairs(tm, pairs, elem=6):
    a, b = [p[0] for p in pairs], [p[1] for p in pairs]
    exp = np.asarray(oracle.redistribution_cost_batch(W.batch(a), W.batch(b), elem))
    got = tm.tm_eval_redistribution_batch(W.batch(a), W.batch(b), elem).cpu().numpy()
    assert (got == exp).all()
    k = int(a[0]["lrank"])
    h = huge((6, 5, 4, 3)[:k], 2, 2)
    gen = tm.tm_eval_redistribution_batch(W.batch(a + [h]), W.batch(b + [h]), elem).cpu().numpy()
    assert (gen[:-1] == exp).all() and not gen[-1].any()


def forms(n, seed, k, ext):
    """Random projections of few domains and machines, so that pairs exist."""
    recs = []
    for c in random_forms(40 * n, seed, k, 30):
        c = c.copy()
        c["extent"][:k] = ext
        if int(c["nodes"]) * int(c["gpus"]) in (6, 8, 12) and oracle.validate(c)[0] == 0:
            recs.append(c)
    return recs[:n]


@pytest.mark.parametrize("seed", [1, 2])
def test_matmul_random_forms(tm, seed):
    say("matmul forms", seed)
    check_matmul(tm, list(random_forms(80, seed, 3, 24)))


def test_matmul_shared_coordinates(tm):
    say("matmul, shared coordinates")
    same = W.candidate((10, 6, 8), 4, 4, [split(0, 2)], [(0, B), (0, B), (0, C)])  # cells 0 and 4
    every = W.candidate((10, 6, 8), 8, 8, [], [(0, B), (0, B)])                    # cells 0 and 1
    below = W.candidate((64, 32, 32), 8, 8, [balance_split(0, 9), decompose(2, (2, 4))], [(0, C), (0, B), (1, C), (2, C)])
    fold = lambda d: W.candidate((48, 48, 48), 4, 4, [merge(0, 1), balance_split(0, d), split(1, 1)],  # noqa: E731
                                 [(0, C), (1, B), (2, B)])
    cases = [same, every, below, fold(5), fold(33), W.candidate((70, 60, 50), 32, 32, [decompose(0, (8, 4))], [(0, C), (1, C), (2, C)]),
             W.candidate((41, 47, 43), 2, 3, [balance_split(0, 41), balance_split(0, 47), balance_split(0, 43)],
                         [(0, C), (1, C), (2, B), (1, B), (0, B)])]
    for i, c in enumerate(cases):
        say("case", i)
        check_matmul(tm, [c])
    check_matmul(tm, cases)


@pytest.mark.parametrize("k", [1, 2, 3, 4])
def test_pairs_random_forms(tm, k):
    say("pairs of rank", k)
    ext = [(61,), (37, 53), (19, 17, 23), (7, 11, 5, 13)][k - 1]
    pairs = pairs_of(forms(60, k, k, ext), k)
    assert len(pairs) >= 57
    check_pairs(tm, pairs)
    check_pairs(tm, pairs * 9)  # more workgroups than get 16 waves each


def test_pairs_in_parts(tm):
    say("pairs in parts")
    ext, P = (400, 300, 11), (64, 64)
    f = lambda *fs: W.candidate(ext, P[0], P[1], [merge(0, 1), decompose(0, fs)])  # noqa: E731
    grids = [f(64, 64, 1), f(16, 256, 1), f(128, 4, 8), f(256, 16, 1), f(1, 512, 8)]
    check_pairs(tm, [(a, b) for a in grids for b in grids], 8)
    one = W.candidate(ext, 1, 30, [merge(0, 1), decompose(0, (5, 6))], [(1, B), (0, C)])
    two = W.candidate(ext, 1, 30, [merge(0, 1), decompose(0, (2, 15))], [(1, C), (0, B)])
    check_pairs(tm, [(one, two), (two, one), (one, one)], 8)


def test_pairs_with_many_block_sizes(tm):
    """Nine coprime block sizes along one dim: more than a pair lists."""
    say("pairs with many block sizes")
    a = W.candidate((101, 4), 1, 13585, [balance_split(1, 2), balance_split(2, 3), balance_split(3, 7),
                                         balance_split(4, 17), balance_split(5, 23)], [(0, B)] * 6 + [(1, B)])
    b = W.candidate((101, 4), 1, 13585, [decompose(1, (5, 11, 13, 19))], [(0, B)] * 5)
    check_pairs(tm, [(x, y) for x in (a, b) for y in (a, b)])


def test_more_parts_than_a_grid(tm):
    """16,500 pairs, one of them in 1,024 parts: 2^32 threads in one launch."""
    say("more parts than a grid holds")
    big = [W.candidate((4500, 4400), 512, 8, [merge(0, 1), W.decompose(0, f)]) for f in ((4096, 1), (1, 4096))]
    some = pairs_of(forms(40, 3, 2, (37, 53)), 3)
    pairs = [some[i % len(some)] for i in range(16500)]
    pairs[16400] = tuple(big)
    exp = np.asarray(oracle.redistribution_cost_batch(W.batch([p[0] for p in some]), W.batch([p[1] for p in some]), 8))
    exp = exp[np.arange(len(pairs)) % len(some)]
    exp[16400] = np.asarray(oracle.redistribution_cost_batch(W.batch(big[:1]), W.batch(big[1:]), 8))[0]
    got = tm.tm_eval_redistribution_batch(W.batch([p[0] for p in pairs]), W.batch([p[1] for p in pairs]), 8)
    assert (got.cpu().numpy() == exp).all()
