"""The block-model estimates of simple mappings from their block records, bit-exact against
the oracle: launch ranks 1 to 4, blocks narrower than the halo and empty ones, dims of one
block, and dims with more blocks than there are records at a time (4,096)."""
import sys

import numpy as np
import pytest

import oracle
import oracle.mlp as mlp
import workloads as W
from workloads import balance_split, decompose, merge, swap

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tm():
    import torch
    assert torch.cuda.is_available()
    import paper_2507_17087_amd as m
    m.lib()
    return m


def blocks(ext, P, F, tail=()):
    return W.candidate(ext, P[0], P[1], [merge(0, 1), decompose(0, F)] + list(tail), [(d, W.BLOCK) for d in range(len(F))])


SMALL = [blocks((37,), (2, 6), (12,)), blocks((5,), (4, 4), (16,)), blocks((40, 9), (4, 6), (2, 12)),
         blocks((40, 9), (4, 6), (2, 12), [swap(0, 1)]), blocks((11, 7, 13), (4, 6), (1, 12, 2)),
         blocks((11, 7, 13, 3), (8, 6), (2, 4, 2, 3)), blocks((6, 5, 4, 3), (1, 1), (1, 1, 1, 1)),
         W.candidate((50, 30), 5, 7, [balance_split(0, 3), merge(1, 2)], [(0, W.BLOCK), (1, W.BLOCK)])]
LARGE = [blocks((20000,), (64, 128), (8192,)), blocks((3000,), (64, 128), (8192,)), blocks((9000, 7), (128, 128), (8192, 2)),
         blocks((7, 9000), (128, 128), (2, 8192)), blocks((5000, 3, 2), (41, 300), (4100, 3, 1)),
         blocks((4097,), (17, 241), (4097,))]


@pytest.mark.parametrize("halo", [(1, 1, 1, 1), (4, 3, 0, 2)])
@pytest.mark.parametrize("recs", [SMALL, LARGE, SMALL + LARGE], ids=["small", "large", "both"])
def test_estimates_from_records(tm, recs, halo):
    import torch
    print("[gpu-case] estimates", len(recs), halo, file=sys.stderr, flush=True)
    assert all(oracle.validate(c)[0] == 0 for c in recs)
    p = tm.Plan(len(recs)).load(W.batch(recs), W.stencil(halo, 8))
    got = tm.tm_ranker_block_estimates(p).cpu().numpy()
    exp = np.array([mlp.block_estimates(c, halo[:int(c["lrank"])], oracle.chain_table) for c in recs])
    assert (got == exp).all()
    torch.cuda.synchronize()


def test_estimates_at_an_address_of_8_bytes(tm):
    import torch
    print("[gpu-case] estimates at an address of 8 bytes", file=sys.stderr, flush=True)
    recs = SMALL + [W.candidate((40, 9), 4, 6, [], [(0, W.CYCLIC), (1, W.BLOCK)])]
    p = tm.Plan(len(recs)).load(W.batch(recs), W.stencil((1, 2, 1, 1), 8))
    buf = torch.full((2 * len(recs) + 2,), -1.0, dtype=torch.float64, device="cuda")
    assert buf.data_ptr() % 16 == 0
    assert tm.lib().tm_ranker_block_estimates(p._p, buf.data_ptr() + 8, None) == tm.TM_OK
    torch.cuda.synchronize()
    assert torch.equal(buf[1:-1].view(-1, 2), tm.tm_ranker_block_estimates(p))
    assert float(buf[0]) == -1.0 and float(buf[-1]) == -1.0
