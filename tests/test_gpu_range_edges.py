"""Range search at the edges of its bit-per-pair filter: limits that fall
exactly on distances, an empty or one-point range, a lower limit below FP32's
smallest number, squared limits beyond FP32, leaves of one to 64 points, and
few enough queries that several waves share a slot.  Sets and distances equal
the FP64 oracle's exactly."""
import numpy as np
import pytest

from oracle import knn as ok

pytestmark = pytest.mark.gpu

ROOT2 = float(np.sqrt(2.0))


@pytest.mark.parametrize("lo,hi", [(0.0, 0.0), (0.0, 1.0), (1.0, 1.0), (1.0, ROOT2), (1e-30, 2.0),
                                   (0.0, 1e25), (2.0, 1e25), (0.0, 1e-30)])
@pytest.mark.parametrize("d,leaf", [(2, 1), (3, 20), (3, 33), (3, 64), (5, 32), (12, 32), (20, 7)])
def test_limits_on_distances(lo, hi, d, leaf):
    import torch
    from paper_1304_4327_amd import knn
    rng = np.random.default_rng(d * 100 + leaf)
    ref = rng.integers(0, 4, (333, d)).astype(np.float32)   # duplicates and equal distances
    q = np.concatenate([ref[:50], rng.integers(0, 4, (31, d)).astype(np.float32)])
    rt = knn.knn_build_tree(torch.from_numpy(ref).cuda(), leaf)
    for pts, own in ((q, False), (ref, True)):
        qt = None if own else knn.knn_build_tree(torch.from_numpy(pts).cuda(), leaf)
        off, idx, dist, _ = knn.knn_range_search(rt, qt, lo, hi, exclude_self=own)
        torch.cuda.synchronize()
        off, idx, dist = off.cpu().numpy(), idx.cpu().numpy(), dist.cpu().numpy()
        oo, oi, od2 = ok.range_rows(pts, np.arange(len(pts)), ref, lo, hi, exclude_self=own)
        assert np.array_equal(off, oo)
        for r in range(len(pts)):
            gi, gd = idx[off[r]:off[r + 1]], dist[off[r]:off[r + 1]]
            o = np.argsort(gi)
            assert np.array_equal(gi[o], oi[oo[r]:oo[r + 1]])
            assert np.array_equal(gd[o], np.sqrt(od2[oo[r]:oo[r + 1]]).astype(np.float32))
