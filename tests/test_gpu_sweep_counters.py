"""Counters of the sweep (stride 64, and FP32 at stride 32): every wave's work is
counted, also where the four waves of a workgroup share a pair of query leaves."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _trees(ref, q, leaf=32):
    import torch
    from paper_1304_4327_amd import knn
    return (knn.knn_build_tree(torch.from_numpy(ref).cuda(), leaf),
            knn.knn_build_tree(torch.from_numpy(q).cuda(), leaf))


# without pruning every pair of points is evaluated: one and two query leaves
# spread over all references, whose blocks are dealt to four waves
@pytest.mark.parametrize("d,precision", [(17, "fp32"), (32, "fp32"), (40, "fp32"), (64, "fp32"),
                                         (64, "bf16")])
@pytest.mark.parametrize("n_q", [32, 60])
def test_every_pair_is_counted(d, precision, n_q):
    from paper_1304_4327_amd import knn
    print(f"counters d={d} {precision} n_q={n_q}", flush=True)
    rng = np.random.default_rng(d)
    ref = rng.random((5000, d)).astype(np.float32)
    q = rng.random((n_q, d)).astype(np.float32)
    rt, qt = _trees(ref, q)
    _, _, st = knn.knn_search(rt, qt, 10, bound="none", precision=precision, stats=True)
    assert st["pairs"] == n_q * 5000
    leaves = knn.knn_tree_get_info(rt)["n_leaves"]
    waves = -(-knn.knn_tree_get_info(qt)["n_leaves"] // 2)
    assert st["leaf_tiles"] == st["score_calls"] == waves * leaves
    assert st["inserts"] >= n_q * 10


# ... also where the order of the blocks would end the sweep early: queries in
# one of several clusters, and query leaves of their own workgroups
@pytest.mark.parametrize("d,precision", [(17, "fp32"), (32, "fp32"), (40, "fp32"), (64, "fp32"),
                                         (64, "bf16")])
@pytest.mark.parametrize("n_q", [1, 300, 66_000])
def test_no_bound_prunes_nothing(d, precision, n_q):
    from oracle import knn as ok
    from oracle import parity
    from paper_1304_4327_amd import knn
    print(f"no bound d={d} {precision} n_q={n_q}", flush=True)
    rng = np.random.default_rng(d + n_q)
    centres = rng.uniform(-1000, 1000, (6, d))
    ref = (centres[rng.integers(0, 6, 6000)] + rng.random((6000, d))).astype(np.float32)
    q = (centres[0] + rng.random((n_q, d))).astype(np.float32)
    rt, qt = _trees(ref, q)
    i, x, st = knn.knn_search(rt, qt, 10, bound="none", precision=precision, stats=True)
    assert st["pairs"] == n_q * 6000
    rows = np.arange(0, n_q, max(1, n_q // 100))
    oi, od = ok.knn_rows(q, rows, ref, 10)
    parity.assert_ok(q, ref, 10, i.cpu().numpy(), x.cpu().numpy(), oi, od, rows=rows)
    _, _, st = knn.knn_search(rt, qt, 10, precision=precision, stats=True)
    assert st["pairs"] < n_q * 6000
