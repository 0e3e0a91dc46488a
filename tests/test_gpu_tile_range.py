"""FP32 requests at d = 5 to 16 through the walk with matrix-core tiles (the
walk that a call with counters takes) where centred norms leave FP32's range:
far points among the references and the queries, and coordinates so small that
squares underflow.  The lists are those of the kernel that works on direct
differences (one query per wave), and the oracle's; BF16 requests take the same
tiles."""
import numpy as np
import pytest

from oracle import knn as ok
from test_gpu_sweep_range import check_oracle, far_sets

pytestmark = pytest.mark.gpu


def _search(ref, q, k, leaf, bound="B"):
    import torch
    from paper_1304_4327_amd import knn
    rt = knn.knn_build_tree(torch.from_numpy(ref).cuda(), leaf)
    qt = knn.knn_build_tree(torch.from_numpy(q).cuda(), leaf)
    walk = knn.knn_search(rt, qt, k, bound=bound, stats=True)
    few = knn.knn_search(rt, qt, k, bound="B" if bound == "none" else bound)
    bf16 = knn.knn_search(rt, qt, k, bound=bound, stats=True, precision="bf16") if ref.shape[1] > 8 else walk
    torch.cuda.synchronize()
    return walk, few, bf16


@pytest.mark.parametrize("n_ref,n_q,leaf,k", [(40, 20, 32, 3), (700, 90, 24, 5), (5000, 700, 32, 16)])
@pytest.mark.parametrize("far_ref,far_q", [((1e25,), ()), ((), (1e25,)), ((3e19, -1e30), ()),
                                           ((1e30, 3e38), (1e25, -3e38)), ((1e22,), (1e22, 4e19))])
@pytest.mark.parametrize("d", [5, 8, 13, 16])
def test_far_points(d, far_ref, far_q, n_ref, n_q, leaf, k):
    print(f"tile far d={d} ref={far_ref} q={far_q} {n_ref}x{n_q} leaf={leaf} k={k}", flush=True)
    ref, q = far_sets(n_ref, n_q, d, far_ref, far_q)
    for bound in ("B", "none"):
        walk, few, bf16 = _search(ref, q, k, leaf, bound)
        assert np.array_equal(walk[0].cpu(), few[0].cpu()) and np.array_equal(walk[1].cpu(), few[1].cpu())
        check_oracle(q, ref, k, walk[0], walk[1])
        check_oracle(q, ref, k, bf16[0], bf16[1])


@pytest.mark.parametrize("scale", [1e-14, 1e-18, 1e-20])
@pytest.mark.parametrize("d", [5, 8, 13, 16])
def test_small_coordinates(d, scale):
    rng = np.random.default_rng(d)
    for mixed in (False, True):
        ref = (rng.standard_normal((3000, d)) * scale).astype(np.float32)
        q = (rng.standard_normal((400, d)) * scale).astype(np.float32)
        if mixed:
            ref[1500:] = rng.standard_normal((1500, d))
            q[200:] = rng.standard_normal((200, d))
        print(f"tile small d={d} scale={scale} mixed={mixed}", flush=True)
        walk, few, bf16 = _search(ref, q, 10, 32)
        for got in (walk, few, bf16):
            if scale >= 1e-18:
                check_oracle(q, ref, 10, got[0], got[1])
            else:
                # the smallest squares here are 1e-41, multiples of 1.4e-45: d
                # roundings of half a step, of either candidate, are at most
                # 1.2e-3 of the square
                od = np.sqrt(ok.knn(q, ref, 10)[1])
                np.testing.assert_allclose(got[1].cpu().numpy(), od, rtol=6e-4)
