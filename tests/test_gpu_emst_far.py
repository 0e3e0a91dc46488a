"""Spanning trees of sets in which some points have fewer than a list of
neighbours within FP32's range: their squared distances to all others (or to
all but a few) overflow, so the list search returns entries without an index.
Such a point lists nothing and is decided by the walk in FP64.  Edge for edge
the oracle's."""
import numpy as np
import pytest

from test_gpu_emst import _check, _emst

pytestmark = pytest.mark.gpu


def _with_far_points(n, d, rng, far):
    x = rng.normal(size=(n, d)).astype(np.float32)
    rows = rng.choice(n, len(far), replace=False)
    for r, f in zip(rows, far):
        x[r] += np.float32(f) * rng.normal(size=d).astype(np.float32)
    return np.ascontiguousarray(x)


# one far point; two of which each is the other's nearest; a group of four far
# from the rest and near each other (lists of three entries)
@pytest.mark.parametrize("far", [(1e25,), (1e20, -1e20), (1e30, 1e25, 3e19)])
@pytest.mark.parametrize("n,d,leaf", [(2048, 3, 20), (2500, 1, 64), (3001, 4, 32), (2222, 5, 32),
                                      (2100, 8, 1)])
def test_far_points(far, n, d, leaf):
    print(f"emst far={far} n={n} d={d} leaf={leaf}", flush=True)
    x = _with_far_points(n, d, np.random.default_rng(n + d), far)
    for bound in ("B", "B1"):
        _check(x, _emst(x, leaf, bound=bound))


@pytest.mark.parametrize("n,d,leaf", [(2048, 3, 20), (2300, 8, 32)])
def test_far_group(n, d, leaf):
    rng = np.random.default_rng(n)
    x = rng.normal(size=(n, d)).astype(np.float32)
    at = np.full(d, 1e24, np.float32)
    for i in range(4):  # neighbouring floats: distances about 1e17
        at = np.nextafter(at, np.float32(np.inf))
        x[17 * i + 3] = at
    print(f"emst far group n={n} d={d} leaf={leaf}", flush=True)
    for bound in ("B", "B1"):
        _check(x, _emst(x, leaf, bound=bound))
