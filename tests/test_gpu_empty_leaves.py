"""Reference and query trees of leaf size 1 over a number of points that is not a
power of two: some leaves are empty.  An empty reference leaf holds no candidate
for the matrix-core tiles of the walk."""
import numpy as np
import pytest

from oracle import knn as ok
from oracle import parity

pytestmark = pytest.mark.gpu


def _run(n_ref, n_q, d, k, ref_leaf, q_leaf, bound, **kw):
    import torch
    from paper_1304_4327_amd import knn
    rng = np.random.default_rng(n_ref + d)
    ref = rng.standard_normal((n_ref, d)).astype(np.float32)
    q = rng.standard_normal((n_q, d)).astype(np.float32)
    q[:n_q // 2] = ref[rng.integers(0, n_ref, n_q // 2)]  # also queries on a point
    print(f"empty leaves: {n_ref}x{n_q} d={d} k={k} leaves {ref_leaf} {q_leaf} {bound} {kw}", flush=True)
    rt = knn.knn_build_tree(torch.from_numpy(ref).cuda(), ref_leaf)
    qt = knn.knn_build_tree(torch.from_numpy(q).cuda(), q_leaf)
    i, x, _ = knn.knn_search(rt, qt, k, bound=bound, **kw)
    oi, od = ok.knn(q, ref, k)
    parity.assert_ok(q, ref, k, i.cpu().numpy(), x.cpu().numpy(), oi, od)


@pytest.mark.parametrize("bound", ["B", "none"])
@pytest.mark.parametrize("n_ref,n_q,q_leaf", [(70, 40, 1), (318, 938, 1), (363, 500, 32), (1030, 60, 20)])
@pytest.mark.parametrize("d,k", [(9, 4), (16, 10), (17, 8), (24, 16), (32, 2)])
def test_bf16(bound, n_ref, n_q, q_leaf, d, k):
    import torch
    _run(n_ref, n_q, d, k, 1, q_leaf, bound, precision="bf16")
    leaves = 1
    while -(-n_q // leaves) > q_leaf:
        leaves *= 2
    seed = torch.full((leaves,), 0.5, device="cuda")
    _run(n_ref, n_q, d, k, 1, q_leaf, bound, precision="bf16", seed_radius=seed)


@pytest.mark.parametrize("bound", ["B", "none"])
@pytest.mark.parametrize("n_ref", [2060, 3001])
@pytest.mark.parametrize("d,k", [(5, 4), (8, 10), (13, 16)])
def test_fp32(bound, n_ref, d, k):
    _run(n_ref, 500, d, k, 1, 32, bound, stats=True)
