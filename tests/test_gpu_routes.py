"""The kernels that serve a call beside the plain slot-per-wave walk return what
it returns, ties at the k-th place included: one query per wave (few queries,
d <= 16) against the walk that a call with counters takes (plain, or with
matrix-core tiles at 5 <= d <= 16 with leaves of 17 to 32 points and lists of
up to 16), and the FP32 sweep at d > 32 against the no-alloc entry's walk.  Bit
for bit: the distances are the same numbers and every tie follows the walk's
order."""
import numpy as np
import pytest

from oracle import knn as ok
from oracle import parity
from paper_1304_4327_amd import datagen

pytestmark = pytest.mark.gpu


def _points(kind, n, d, seed):
    rng = np.random.default_rng(seed)
    if kind == "lattice":  # many equal distances
        return rng.integers(0, max(2, round(n ** (1.0 / d))), (n, d)).astype(np.float32)
    x = (rng.standard_normal((n, d)) * rng.uniform(0.2, 3.0, d)).astype(np.float32)
    if kind == "twice":    # every point two times: ties in pairs
        x[n // 2:2 * (n // 2)] = x[:n // 2]
    return x


def _trees(ref, q, leaf):
    import torch
    from paper_1304_4327_amd import knn
    rt = knn.knn_build_tree(torch.from_numpy(ref).cuda(), leaf)
    return rt, None if q is None else knn.knn_build_tree(torch.from_numpy(q).cuda(), leaf)


# reference sizes: one leaf; one, two and three steps of six levels; k from 1
# to the longest list of the kernel (62 with the query's own point)
@pytest.mark.parametrize("n_ref,leaf,k", [(30, 32, 7), (700, 32, 1), (3000, 20, 62), (3000, 64, 10),
                                          (9000, 2, 5), (60_000, 16, 16), (20_000, 32, 10),
                                          (5000, 24, 14)])
@pytest.mark.parametrize("d,kind", [(1, "random"), (2, "lattice"), (3, "twice"), (4, "random"),
                                    (5, "random"), (8, "twice"), (13, "random"), (16, "twice")])
def test_one_query_per_wave_equals_the_walk(n_ref, leaf, k, d, kind):
    import torch
    from paper_1304_4327_amd import knn
    for n_q in (0, 1, 333):
        print(f"few: n_ref={n_ref} n_q={n_q} d={d} k={k} leaf={leaf} {kind}", flush=True)
        ref = _points(kind, n_ref, d, n_ref + d)
        q = _points(kind, n_q, d, d) if n_q else None
        if q is None and n_ref > 32768:
            continue
        kk = k - 1 if q is None and k == 62 else k
        if q is not None and kind == "twice":
            m = min(n_q, n_ref) // 2
            q[:m] = ref[:m]  # distance 0, two times
        rt, qt = _trees(ref, q, leaf)
        got = knn.knn_search(rt, qt, kk, exclude_self=q is None)
        want = knn.knn_search(rt, qt, kk, exclude_self=q is None, stats=True)
        torch.cuda.synchronize()
        assert torch.equal(got[1], want[1])
        # a lattice can hold more equal distances than the lanes past the
        # k-th entry: then only the distances are compared
        if kind != "lattice":
            assert torch.equal(got[0], want[0])


@pytest.mark.parametrize("n_ref,n_q,leaf,k", [(40, 5, 32, 7), (900, 70, 16, 1), (5000, 400, 32, 50),
                                              (5000, 900, 20, 62), (3000, 0, 32, 16),
                                              (2100, 66_000, 32, 8)])
@pytest.mark.parametrize("d,kind", [(33, "random"), (64, "twice")])
def test_fp32_sweep_equals_the_walk(n_ref, n_q, leaf, k, d, kind):
    """The FP32 sweep (parts of a workgroup and whole workgroups) against the
    walk of the no-alloc entry, and against the oracle."""
    import torch
    from paper_1304_4327_amd import knn
    ref = _points(kind, n_ref, d, n_ref)
    q = _points(kind, n_q, d, 7) if n_q else None
    if q is not None and kind == "twice":
        m = min(n_q, n_ref) // 2
        q[:m] = ref[:m]
    rt, qt = _trees(ref, q, leaf)
    nq = n_q or n_ref
    print(f"pair: n_ref={n_ref} n_q={n_q} d={d} k={k} leaf={leaf} {kind}", flush=True)
    got = knn.knn_search(rt, qt, k, exclude_self=q is None)
    out = (torch.empty((nq, k), dtype=torch.int64, device="cuda"),
           torch.empty((nq, k), dtype=torch.float32, device="cuda"))
    want = knn.knn_search_noalloc(rt, qt, k, out, exclude_self=q is None)
    torch.cuda.synchronize()
    assert torch.equal(got[1], want[1]) and torch.equal(got[0], want[0])
    if kind == "random":
        rows = np.arange(0, nq, max(1, nq // 200))
        x = ref if q is None else q
        oi, od = ok.knn_rows(x, rows, ref, k, exclude_self=q is None)
        parity.assert_ok(x, ref, k, got[0].cpu().numpy(), got[1].cpu().numpy(), oi, od, rows=rows)


# the walk's blocks of five levels: trees of 0 to 11 levels, so that the first
# block has every size; with counters the slot-per-wave walk serves the call
@pytest.mark.parametrize("levels", [0, 1, 2, 3, 4, 5, 6, 9, 10, 11])
@pytest.mark.parametrize("d,leaf,k", [(1, 1, 3), (3, 2, 10), (4, 32, 5), (8, 32, 10), (8, 7, 20),
                                      (12, 32, 4), (16, 24, 15)])
def test_walk_blocks_of_every_height(levels, d, leaf, k):
    import torch
    from paper_1304_4327_amd import knn
    n = max(k + 1, (leaf << levels) - 1)
    if n > 40_000:
        n = 40_000
    for kind in ("random", "twice"):
        ref, q = _points(kind, n, d, n + d), _points(kind, 300, d, d)
        rt, qt = _trees(ref, q, leaf)
        walk = knn.knn_search(rt, qt, k, stats=True)
        few = knn.knn_search(rt, qt, k)
        torch.cuda.synchronize()
        assert torch.equal(walk[0], few[0]) and torch.equal(walk[1], few[1])


# the same sweep at stride 32
@pytest.mark.parametrize("n_ref,n_q,leaf", [(40, 5, 32), (1000, 1, 20), (1000, 700, 32),
                                            (5000, 0, 16), (33_000, 900, 32), (3000, 20_000, 31)])
@pytest.mark.parametrize("d,k,kind", [(17, 1, "random"), (20, 8, "twice"), (24, 16, "random"),
                                      (32, 31, "twice"), (32, 10, "twice"), (30, 7, "random")])
def test_fp32_sweep_at_stride_32(n_ref, n_q, leaf, d, k, kind):
    test_fp32_sweep_equals_the_walk(n_ref, n_q, leaf, k, d, kind)


@pytest.mark.parametrize("k", [6, 39, 51, 63])
def test_fp32_sweep_at_stride_32_long_lists(k):
    test_fp32_sweep_equals_the_walk(4000, 300, 32, k, 27, "random")
