"""Kernel density sums over trees of every height around the five levels that
the walk scores at once (one leaf, a first block of one to five levels, one to
three blocks), with empty leaves and duplicates, against the FP64 oracle: the
budget is that of test_gpu_kde.  Leave-one-out only with exact sums: a node
that is approximated counts all of its points, the query's own among them.
The bandwidth keeps every kernel value a normal FP32 number."""
import numpy as np
import pytest

from test_gpu_kde import _check, _kde

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 20])
@pytest.mark.parametrize("n,leaf", [(1, 1), (2, 1), (3, 1), (17, 1), (32, 1), (33, 1), (60, 1),
                                    (65, 2), (1025, 1), (2500, 1), (3000, 64)])
def test_heights(n, leaf, d):
    rng = np.random.default_rng(n * 10 + d)
    ref = rng.normal(size=(n, d)).astype(np.float32)
    ref[n // 2:n // 2 + 5] = ref[0]
    q = rng.normal(size=(70, d)).astype(np.float32)
    for pts, own in ((q, False), (None, True)):
        for eps in (0.0,) if own else (0.0, 0.02 * n):
            f, st = _kde(ref, pts, 4.0, eps, leaf, stats=True, self_mode=own)
            _check(ref, pts, 4.0, eps, f, self_mode=own)
            if eps == 0.0:
                assert st["inserts"] == 0 and st["pairs"] == n * (n if own else len(q))
