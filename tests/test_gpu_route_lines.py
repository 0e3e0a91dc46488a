"""Calls on both sides of the lines that choose a kernel by the number of
references and queries return the same neighbours: those of the call with
counters (the slot-per-wave walk) or of the no-alloc entry, and the oracle's."""
import numpy as np
import pytest

from oracle import knn as ok
from oracle import parity

pytestmark = pytest.mark.gpu


def _check(n_ref, n_q, d, k, leaf=32):
    import torch
    from paper_1304_4327_amd import knn
    print(f"lines: {n_ref}x{n_q} d={d} k={k}", flush=True)
    rng = np.random.default_rng(n_ref + n_q)
    ref = rng.standard_normal((n_ref, d)).astype(np.float32)
    q = rng.standard_normal((n_q, d)).astype(np.float32)
    rt = knn.knn_build_tree(torch.from_numpy(ref).cuda(), leaf)
    qt = knn.knn_build_tree(torch.from_numpy(q).cuda(), leaf)
    got = knn.knn_search(rt, qt, k)
    counted = knn.knn_search(rt, qt, k, stats=True)
    out = (torch.empty((n_q, k), dtype=torch.int64, device="cuda"),
           torch.empty((n_q, k), dtype=torch.float32, device="cuda"))
    fixed = knn.knn_search_noalloc(rt, qt, k, out)
    torch.cuda.synchronize()
    for other in (counted, fixed):
        assert torch.equal(got[0], other[0]) and torch.equal(got[1], other[1])
    rows = np.arange(0, n_q, max(1, n_q // 200))
    oi, od = ok.knn_rows(q, rows, ref, k)
    parity.assert_ok(q, ref, k, got[0].cpu().numpy(), got[1].cpu().numpy(), oi, od, rows=rows)


# matrix-core tiles for FP32 requests
@pytest.mark.parametrize("n_ref", [2047, 2048])
@pytest.mark.parametrize("n_q", [500, 71_000])
@pytest.mark.parametrize("d", [5, 8, 9, 16])
def test_tiles_by_references(n_ref, n_q, d):
    _check(n_ref, n_q, d, 10)


# one query per wave: the last number of queries it takes and the next
def _most(n_ref, d, k):
    most = 65536 + n_ref // (6 if d <= 4 else 2 if d <= 8 else 8)
    if k > 16:
        return most
    line = {1: 24576 + n_ref // 8, 2: min(most, 32768 + n_ref // 2)}.get(d, most)
    return min(line, 16384 + 48 * n_ref)


@pytest.mark.parametrize("n_ref", [100, 3000, 20_000])
@pytest.mark.parametrize("d,k", [(1, 6), (2, 6), (2, 17), (3, 6), (8, 6), (12, 16)])
def test_one_query_per_wave_by_queries(n_ref, d, k):
    for more in (0, 1):
        _check(n_ref, _most(n_ref, d, k) + more, d, k)


# the sweep for FP32 requests
@pytest.mark.parametrize("n_ref", [2999, 3000])
@pytest.mark.parametrize("n_q", [1, 500, 20_000])
@pytest.mark.parametrize("d", [17, 32, 33, 64])
def test_sweep_by_references(n_ref, n_q, d):
    for k in (10, 50):
        _check(n_ref, n_q, d, k)
