"""Calls that find no memory for part of their scratch: the FP32 sweep's
operands and the spanning tree's neighbour lists are left out and the walks
serve the call, with the same answer; anything else reports KNN_E_OOM, and the
next call is served as usual."""
import numpy as np
import pytest

from oracle import knn as ok

pytestmark = pytest.mark.gpu


def _failing(after, call):
    """call() with the after-th allocation failing: (its result or None, whether
    the failure happened)."""
    from paper_1304_4327_amd import knn
    lib = knn.load()
    lib.knn_debug_fail_alloc(after)
    try:
        out = call()
    except knn.KnnError as e:
        assert e.status == knn.KNN_E_OOM
        out = None
    return out, lib.knn_debug_fail_alloc(-1) < 0


@pytest.mark.parametrize("d", [24, 64])
@pytest.mark.parametrize("n_q", [300, 5000])
def test_fp32_sweep_without_its_operands(d, n_q):
    import torch
    from paper_1304_4327_amd import knn
    rng = np.random.default_rng(d)
    ref = torch.from_numpy(rng.standard_normal((6000, d)).astype(np.float32)).cuda()
    q = torch.from_numpy(rng.standard_normal((n_q, d)).astype(np.float32)).cuda()
    rt, qt = knn.knn_build_tree(ref, 32), knn.knn_build_tree(q, 32)
    want = knn.knn_search(rt, qt, 10)
    served = 0
    for after in range(40):
        print(f"sweep d={d} n_q={n_q} allocation {after}", flush=True)
        got, failed = _failing(after, lambda: knn.knn_search(rt, qt, 10))
        torch.cuda.synchronize()
        if got is not None:
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        if not failed:
            break
        served += got is not None
    else:
        pytest.fail("more allocations than a search makes")
    assert served == 8  # the eight operand arrays


@pytest.mark.parametrize("n,d", [(2500, 3), (2300, 8)])
def test_spanning_tree_without_its_lists(n, d):
    import torch
    from paper_1304_4327_amd import knn
    x = np.random.default_rng(n).standard_normal((n, d)).astype(np.float32)
    t = knn.knn_build_tree(torch.from_numpy(x).cuda(), 32)
    u, v, _ = ok.emst(x)
    want = ok.edge_set(u, v)
    served = 0
    for after in range(60):
        print(f"emst n={n} d={d} allocation {after}", flush=True)
        got, failed = _failing(after, lambda: knn.knn_emst(t))
        torch.cuda.synchronize()
        if got is not None:
            assert np.array_equal(ok.edge_set(got[0].cpu().numpy(), got[1].cpu().numpy()), want)
        if not failed:
            break
        served += got is not None
    else:
        pytest.fail("more allocations than a spanning tree makes")
    assert served >= 7  # the four list arrays and the list search's three


@pytest.mark.parametrize("n,d", [(20, 3), (30_000, 3), (30_000, 40)])
def test_build_without_scratch(n, d):
    import torch
    from paper_1304_4327_amd import knn
    x = torch.from_numpy(np.random.default_rng(n).standard_normal((n, d)).astype(np.float32)).cuda()
    for after in range(60):
        print(f"build n={n} d={d} allocation {after}", flush=True)
        t, failed = _failing(after, lambda: knn.knn_build_tree(x, 32))
        assert (t is None) == failed
        if t is not None:
            t.close()
            break
    else:
        pytest.fail("more allocations than a build makes")
