"""The gradient's tiles at their edges: one row, part tiles of 16 and 32 rows, the change
from 16-row to 32-row tiles (above 4,096 rows), one and several row ranges with a short
last one; the same inputs give the same bits; a batch after a larger one."""
import numpy as np
import pytest

from oracle import mlp
from test_gpu_ranker import _determined_rows, _elementwise_ok, say, tm  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 16, 17, 33, 511, 513, 4096, 4097, 9001])
def test_gradient_tiles(tm, rows):  # noqa: F811
    import torch
    say("gradient tiles", rows)
    r = tm.Ranker(seed=rows)
    rng = np.random.default_rng(rows)
    p = r.get_params().cpu().numpy().astype(np.float64)
    X = rng.uniform(-1, 1, size=(4 * rows + 64, mlp.F)).astype(np.float32)
    X = _determined_rows(p, X.astype(np.float64), rows).astype(np.float32)
    T = rng.normal(0, 1, size=(rows, mlp.O)).astype(np.float32)
    xd, td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    g = r.grad(xd, td)
    # a larger batch in between leaves nothing behind in the buffers
    r.grad(torch.ones(rows + 100, mlp.F, device="cuda"), torch.zeros(rows + 100, mlp.O, device="cuda"))
    assert torch.equal(g, r.grad(xd, td))
    g = g.cpu().numpy().astype(np.float64)
    _, ref = mlp.loss_and_grad(p, X.astype(np.float64), T.astype(np.float64), "bf16")
    L = mlp.layout()
    ok = [_elementwise_ok(g[a:b], ref[a:b], k) for k, (a, b) in
          ((k, L[k]) for k in ("w1", "b1", "w2", "b2", "w3", "b3", "w4", "b4"))]
    assert all(ok)
