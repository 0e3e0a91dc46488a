"""Spanning trees through the neighbour lists, at their edges: the smallest set
that gets lists, more than a list of duplicates, equal lengths on a lattice,
coordinates whose squared distances leave FP32's range at either end, and
clusters smaller and larger than a list.  Edge for edge the oracle's."""
import numpy as np
import pytest

from test_gpu_emst import _check, _emst

pytestmark = pytest.mark.gpu


def _points(kind, n, d, rng):
    x = rng.normal(size=(n, d)).astype(np.float32)
    if kind == "duplicates":
        x[rng.integers(0, n, n // 2)] = x[:n // 2][rng.integers(0, 40, n // 2)]
    elif kind == "lattice":
        x = rng.integers(0, 12, (n, d)).astype(np.float32)
    elif kind == "huge":
        x *= np.float32(3e18)
    elif kind == "tiny":
        x *= np.float32(1e-18)
    elif kind == "clusters":
        sizes = rng.choice([3, 9, 10, 11, 12, 40], n)
        x = x * np.float32(1e-3) + (np.repeat(np.arange(n), sizes)[:n, None] * 7).astype(np.float32)
    return np.ascontiguousarray(x, dtype=np.float32)


@pytest.mark.parametrize("kind", ["normal", "duplicates", "lattice", "huge", "tiny", "clusters"])
@pytest.mark.parametrize("n,d,leaf", [(2047, 3, 20), (2048, 3, 20), (2500, 1, 64), (2600, 2, 7),
                                      (3001, 4, 32), (2222, 5, 32), (2100, 8, 1)])
def test_lists(kind, n, d, leaf):
    rng = np.random.default_rng(n + d)
    ref = _points(kind, n, d, rng)
    for bound in ("B", "B1"):
        _check(ref, _emst(ref, leaf, bound=bound))
