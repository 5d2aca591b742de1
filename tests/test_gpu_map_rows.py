"""Processor maps where a 16-byte store meets the rows' ends, bit-exact against the oracle:
rows of 1 to 5 points and of no multiple of 4, rows longer than a workgroup's block, blocks
of 3, 4 and 5 points along the last dim, several projections of it, cyclic ones, owner
tables on both sides of the one-wave limit, output at every offset from 16-byte alignment,
and one launch that fits a batch of different domains."""
import random
import sys

import numpy as np
import pytest

import oracle
import workloads as W
from workloads import decompose, merge

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


def grid(ext, F, proj):
    """Final dims F[0] x F[1] over ext, projected as given."""
    return W.candidate(ext, F[0], F[1], [], proj)


CASES = [((n, L), F, [(0, p), (1, q)])
         for n, L in [(1, 1), (700, 1), (513, 2), (5, 3), (1000, 5), (257, 7), (33, 31), (3, 1021), (7, 1024),
                      (2, 4099), (3, 16387)]
         for F in [(2, 3), (4, 8)] for p, q in [(B, B), (C, B), (B, C)]]
CASES += [((9, 3 * s + d), (2, s), [(0, B), (1, B)]) for s in (3, 7, 64) for d in (0, s - 1, s, s + 1, 2 * s)]
CASES += [((40, 30), (3, 4), [(1, B), (1, B)]), ((40, 50), (3, 4), [(1, B), (1, C)]), ((61, 29), (3, 4), [(0, B), (0, C)]),
          ((17, 11, 13), (4, 3), [(0, B), (2, B)]), ((5, 7, 3, 9), (2, 5), [(1, C), (3, B)]),
          ((300, 200), (2048, 1), [(0, B), (1, B)]), ((300, 200), (2049, 1), [(1, C), (0, B)]),
          ((64, 9001), (2, 2048), [(0, B), (1, B)]), ((3, 5000000), (2, 8), [(0, B), (1, B)])]


def test_maps_of_every_row_form(tm):
    for i, (ext, F, proj) in enumerate(CASES):
        c = grid(ext, F, proj)
        say("map", i, ext, F, proj)
        got = tm.tm_proc_map(c).cpu().numpy()
        assert (got == oracle.proc_map(c)).all(), (ext, F, proj)


@pytest.mark.parametrize("wide", [False, True])
def test_unaligned_output_of_one_launch(tm, wide):
    import torch
    say("unaligned maps: wide table", wide)
    forms = [c for c in CASES if c[0][0] * c[0][1] < 20000 and len(c[0]) == 2][::5]
    recs = [grid(*f) for f in forms] + ([grid((300, 200), (2048, 2), [(0, B), (1, B)])] if wide else [])
    cands, n = W.batch(recs), len(recs)
    plan = tm.Plan(n).load(cands, W.stencil((1, 1), 8))
    out = torch.empty((n, 4), dtype=torch.int64, device="cuda")
    best = torch.empty(1, dtype=torch.int64, device="cuda")
    plan.run(out, best)
    points = max(int(np.prod(r["extent"][: int(r["lrank"])])) for r in recs)
    for i, r in enumerate(recs):
        exp = oracle.proc_map(r).ravel()
        buf = torch.full((points + 8,), -7, dtype=torch.int32, device="cuda")
        a = 1 + i % 4
        idx = torch.tensor([i], dtype=torch.int64, device="cuda")
        plan.materialize(buf[a:a + points], d_index=idx)
        got = buf.cpu().numpy()
        assert (got[a:a + exp.size] == exp).all(), forms[i] if i < len(forms) else "wide"
        assert (got[:a] == -7).all() and (got[a + exp.size:] == -7).all()
