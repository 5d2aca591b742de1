"""Batches with a few candidates whose tables exceed the words of the common launch: the
evaluation takes two launches, the selection comes after both.  The number of launches is
counted over a HIP runtime of host memory, the rows are compared on the GPU."""
import sys

import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_groups import random_forms
from test_plan_failures_cpu import HEAD, over_host_memory
from workloads import balance_split, decompose, merge

# one-wave workgroups (largest common launch 2,048 words), four-wave ones (8,192), and so few
# candidates that a single launch would have selected
CASES = [(4200, 64, 0), (600, 2500, 0), (60, 2500, 1 << 20)]


def batch(n, g):
    """Of n candidates every 50th or so has a table of 4 g words, once folded."""
    forms = random_forms(60, 5, 2, 20)
    big = W.batch([W.candidate((70, 3 * g), g, 4, [merge(0, 1), decompose(0, (4, g))]),
                   W.candidate((2 * g, 30), g, 4, [merge(0, 1), decompose(0, (g, 4)), merge(0, 1), balance_split(0, 2 * g + 3)])])
    if g == 64:
        big["nodes"], big["ops"][0]["f"][1] = 1024, (64, 64, 1, 1)
        big["ops"][1]["f"][1] = (2048, 2, 1, 1)
    cands = forms[np.arange(n) % len(forms)]
    at = np.arange(7, n, max(1, min(n // 9, 50)))
    cands[at] = big[np.arange(len(at)) % 2]
    return cands, W.stencil((1, 1), 8)


@pytest.mark.parametrize("n, g, cells", CASES)
def test_launches(tmp_path, n, g, cells):
    over_host_memory(tmp_path, HEAD + f"""
sys.path.insert(0, "tests")
from test_two_launches import batch
c, st = batch({n}, {g})
assert L.tm_plan_create({n}, 1, ctypes.byref(p)) == tm.TM_OK
assert L.tm_plan_load(p, c.ctypes.data, {n}, st.ctypes.data, {cells}, None) == tm.TM_OK, L.tm_last_error()
out, at = np.zeros(({n}, 4), np.int64), launches.value
assert run() == tm.TM_OK
assert launches.value - at == 3, launches.value - at
print("done")
""")


@pytest.mark.gpu
@pytest.mark.parametrize("n, g, cells", CASES)
def test_rows(n, g, cells):
    import torch
    import paper_2507_17087_amd as tm
    print("[gpu-case] two launches of", n, file=sys.stderr, flush=True)
    cands, st = batch(n, g)
    exp = oracle.stencil_cost_batch(cands, st)
    plan = tm.Plan(n, 1)
    plan.load(cands, st, cells_per_item=cells)
    out = torch.full((n, 4), -1, dtype=torch.int64, device="cuda")
    best = torch.empty(1, dtype=torch.int64, device="cuda")
    for _ in range(2):
        plan.run(out, best)
        assert (out.cpu().numpy() == exp).all()
        assert int(best.cpu()[0]) == oracle.select_best(exp)
    plan.close()
