"""Matrix-core tiles of the walk where their margin lets most rows through: sets
of a few tight clusters far apart, so that some query leaves span the gap
between two of them and lie far from the centre their tiles are taken about.
The FP32 filter that then joins the products, or takes their place, returns the
lists of the kernel on direct differences, bit for bit, and the oracle's."""
import numpy as np
import pytest

from oracle import knn as ok
from oracle import parity

pytestmark = pytest.mark.gpu


def _clusters(n, d, centres, spread, seed):
    rng = np.random.default_rng(seed)
    c = rng.integers(0, len(centres), n)
    return (centres[c] + spread * rng.standard_normal((n, d))).astype(np.float32)


# leaves that fill their slots and leaves that do not (30 and 21 of 32 points);
# clusters of fewer points than a leaf and of many leaves
@pytest.mark.parametrize("n_ref,n_q,leaf,clusters", [(5000, 1000, 32, 7), (7681, 900, 30, 300),
                                                     (10_752, 2500, 21, 40)])
@pytest.mark.parametrize("d", [5, 6, 8, 9, 13, 16])
@pytest.mark.parametrize("k", [1, 10, 16])
def test_tiles_between_clusters(d, n_ref, n_q, leaf, clusters, k):
    import torch
    from paper_1304_4327_amd import knn
    print(f"loose: d={d} {n_ref}x{n_q} leaf={leaf} clusters={clusters} k={k}", flush=True)
    centres = np.random.default_rng(clusters).uniform(-1000, 1000, (clusters, d))
    ref, q = _clusters(n_ref, d, centres, 1.0, 1), _clusters(n_q, d, centres, 1.0, 2)
    rt = knn.knn_build_tree(torch.from_numpy(ref).cuda(), leaf)
    qt = knn.knn_build_tree(torch.from_numpy(q).cuda(), leaf)
    walk = knn.knn_search(rt, qt, k, stats=True)
    few = knn.knn_search(rt, qt, k)
    torch.cuda.synchronize()
    assert torch.equal(walk[0], few[0]) and torch.equal(walk[1], few[1])
    rows = np.arange(0, n_q, 7)
    oi, od = ok.knn_rows(q, rows, ref, k)
    parity.assert_ok(q, ref, k, walk[0].cpu().numpy(), walk[1].cpu().numpy(), oi, od, rows=rows)
    if d > 8:
        b, bd, _ = knn.knn_search(rt, qt, k, precision="bf16", stats=True)
        parity.assert_ok(q, ref, k, b.cpu().numpy(), bd.cpu().numpy(), oi, od, rows=rows)
