"""FP32 requests at d = 17 to 64 (the sweep, whose filter is a BF16 product
centred on blocks of leaves) where centred norms leave FP32's range: a few
points far from the rest, whose squared distances overflow, and coordinates so
small that they underflow.  Every query gets the neighbours that the walk over
direct differences finds (the no-alloc entry), bit for bit, and the oracle's;
where fewer than k squared distances are finite the rest are -1 and +inf."""
import numpy as np
import pytest

from oracle import knn as ok
from oracle import parity

pytestmark = pytest.mark.gpu

FLT_MAX = float(np.finfo(np.float32).max)


def far_sets(n_ref, n_q, d, far_ref, far_q, seed=3):
    """Ordinary points with some moved far out; the first far query lies next
    to the first far reference (a finite squared distance)."""
    rng = np.random.default_rng(seed)
    ref = rng.standard_normal((n_ref, d)).astype(np.float32)
    q = rng.standard_normal((n_q, d)).astype(np.float32)
    sign = np.where(rng.random((8, d)) < 0.5, -1, 1).astype(np.float32)
    rows_r = rng.choice(n_ref, len(far_ref), replace=False)
    rows_q = rng.choice(n_q, len(far_q), replace=False)
    for i, f in enumerate(far_ref):
        ref[rows_r[i]] = np.float32(f) * sign[i]
    for i, f in enumerate(far_q):
        q[rows_q[i]] = np.float32(f) * sign[i]
    if len(far_q) and len(far_ref):
        q[rows_q[0]] = np.nextafter(ref[rows_r[0]], np.float32(0))
    return ref, q


def check_oracle(q, ref, k, idx, dist):
    gi, gd = idx.cpu().numpy(), dist.cpu().numpy()
    oi, od = ok.knn(q, ref, k)
    near = np.nonzero(od[:, k - 1] < 1e38)[0]
    assert len(near) > 0
    parity.assert_ok(q, ref, k, gi, gd, oi[near], od[near], rows=near)
    for r in np.nonzero(od[:, k - 1] >= 1e38)[0]:
        fin, over = od[r] < 0.99 * FLT_MAX, od[r] > 1.01 * FLT_MAX
        np.testing.assert_allclose(gd[r][fin], np.sqrt(od[r][fin]), rtol=1e-6)
        assert np.all(gi[r][over] == -1) and np.all(np.isinf(gd[r][over]))


def _both(ref, q, k, leaf, bound="B", precision="fp32"):
    import torch
    from paper_1304_4327_amd import knn
    rt = knn.knn_build_tree(torch.from_numpy(ref).cuda(), leaf)
    qt = knn.knn_build_tree(torch.from_numpy(q).cuda(), leaf)
    got = knn.knn_search(rt, qt, k, bound=bound, precision=precision)
    out = (torch.empty((len(q), k), dtype=torch.int64, device="cuda"),
           torch.empty((len(q), k), dtype=torch.float32, device="cuda"))
    want = knn.knn_search_noalloc(rt, qt, k, out, bound=bound)
    torch.cuda.synchronize()
    return got, want


# references of several blocks (1024 points at leaf 32), and of one; query
# leaves shared by a workgroup's waves and one pair a wave
@pytest.mark.parametrize("n_ref,n_q,leaf,k", [(700, 90, 32, 5), (5000, 300, 24, 10),
                                              (4000, 66_000, 32, 16)])
@pytest.mark.parametrize("far_ref,far_q", [((1e25,), ()), ((), (1e25,)), ((3e19, -1e30), ()),
                                           ((1e30, 3e38), (1e25, -3e38)), ((1e22,), (1e22, 4e19))])
@pytest.mark.parametrize("d", [17, 32, 33, 64])
def test_far_points(d, far_ref, far_q, n_ref, n_q, leaf, k):
    print(f"sweep far d={d} ref={far_ref} q={far_q} {n_ref}x{n_q} leaf={leaf} k={k}", flush=True)
    ref, q = far_sets(n_ref, n_q, d, far_ref, far_q)
    got, want = _both(ref, q, k, leaf)
    assert np.array_equal(got[0].cpu(), want[0].cpu()) and np.array_equal(got[1].cpu(), want[1].cpu())
    if n_q <= 300:
        check_oracle(q, ref, k, got[0], got[1])


# coordinates of one small scale, and a small cloud among ordinary points
@pytest.mark.parametrize("scale", [1e-14, 1e-18, 1e-20, 1e-21])
@pytest.mark.parametrize("d", [17, 24, 32, 64])
def test_small_coordinates(d, scale):
    rng = np.random.default_rng(d)
    for mixed in (False, True):
        ref = (rng.standard_normal((3000, d)) * scale).astype(np.float32)
        q = (rng.standard_normal((400, d)) * scale).astype(np.float32)
        if mixed:
            ref[1500:] = rng.standard_normal((1500, d))
            q[200:] = rng.standard_normal((200, d))
        print(f"sweep small d={d} scale={scale} mixed={mixed}", flush=True)
        got, want = _both(ref, q, 10, 32)
        if scale < 1e-20:
            # squared distances of 1e-41 are multiples of 1.4e-45: d roundings
            # of half a step are 4.5e-3 of the square, and the lists compare
            # squares, so either kernel may prefer a point that much farther
            od = np.sqrt(ok.knn(q, ref, 10)[1])
            for x in (got, want):
                np.testing.assert_allclose(x[1].cpu().numpy(), od, rtol=2.5e-3)
            continue
        assert np.array_equal(got[1].cpu(), want[1].cpu())
        # (an ordinary query is at one distance from the whole cloud: more ties
        # than the sweep's lists have spare entries)
        n = 200 if mixed else 400
        assert np.array_equal(got[0][:n].cpu(), want[0][:n].cpu())
        check_oracle(q, ref, 10, got[0], got[1])


# more blocks than the sweep sorts (it goes outward in tree order then)
@pytest.mark.parametrize("far_ref,far_q", [((), ()), ((1e25, -1e30), (1e25,))])
@pytest.mark.parametrize("d", [20, 64])
def test_blocks_in_tree_order(d, far_ref, far_q):
    print(f"sweep unsorted d={d} {far_ref} {far_q}", flush=True)
    ref, q = far_sets(70_000, 200, d, far_ref, far_q)
    got, want = _both(ref, q, 10, 1)
    assert np.array_equal(got[0].cpu(), want[0].cpu()) and np.array_equal(got[1].cpu(), want[1].cpu())
    check_oracle(q, ref, 10, got[0], got[1])
