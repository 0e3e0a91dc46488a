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


# the largest k-th distance of an empty query leaf is 0, in every kernel that
# serves the call
@pytest.mark.parametrize("d,precision", [(3, "fp32"), (8, "fp32"), (16, "fp32"), (16, "bf16"), (24, "fp32"),
                                         (24, "bf16"), (64, "fp32"), (64, "bf16")])
@pytest.mark.parametrize("n_ref,n_q", [(300, 70), (4000, 900)])
def test_kth_distance_of_an_empty_query_leaf(d, precision, n_ref, n_q):
    import torch
    from paper_1304_4327_amd import knn
    print(f"empty query leaves: {n_ref}x{n_q} d={d} {precision}", flush=True)
    rng = np.random.default_rng(d)
    ref = rng.standard_normal((n_ref, d)).astype(np.float32)
    q = rng.standard_normal((n_q, d)).astype(np.float32)
    rt = knn.knn_build_tree(torch.from_numpy(ref).cuda(), 32)
    qt = knn.knn_build_tree(torch.from_numpy(q).cuda(), 1)
    a = knn.tree_arrays(qt)
    first = a["info"]["first_leaf"]
    count, start = a["count"][first:], a["start"][first:]
    assert (count == 0).any() and count.max() == 1
    kth = torch.full((len(count),), -1.0, device="cuda")
    _, x, _ = knn.knn_search(rt, qt, 5, precision=precision, leaf_kth_out=kth)
    torch.cuda.synchronize()
    x, kth = x.cpu().numpy(), kth.cpu().numpy()
    assert np.all(kth[count == 0] == 0.0)
    rows = a["perm"][start[count == 1]]
    np.testing.assert_array_equal(kth[count == 1], x[rows, 4])
