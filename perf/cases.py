"""Performance cases: the calls a program makes to this library, over the
range of sizes, dimensions and options it is used with.

``listed()`` names the fixed cases, ``draw(rng)`` gives further ones of the
same ranges.  ``prepare`` makes what a program holds before the call (points
on the GPU, prebuilt trees where such a program keeps them), ``run`` is one
pass through the public entry points, ``work`` the bytes and operations the
pass cannot do without, ``exact`` the FP64 answer where brute force is
affordable.

Point sets follow the recipes of ``paper_1304_4327_amd.datagen`` (uniform,
Gaussian mixtures with equal or Zipf weights, noisy manifolds), drawn on the
GPU.
"""
from __future__ import annotations

import math

import torch

from paper_1304_4327_amd import knn

DEV = "cuda"


# --------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------
def listed():
    return [
        # an online lookup: a few hundred new points against a tree that the
        # service keeps (latency; the query tree is built inside the call)
        dict(name="lookup_257_d3", op="points", data="gmm", d=3, n_ref=100_000, n_query=257, k=8,
             leaf=32, precision="fp32"),
        # the smallest whole job: a neighbour graph of a small point cloud
        # (normals, outlier scores), every call a new cloud
        dict(name="self_10k_d3_k5", op="all", data="uniform", d=3, n_ref=10_000, n_query=0, k=5,
             leaf=20, precision="fp32"),
        # the headline: registration-sized clouds against each other
        dict(name="pair_1m_d3_k10", op="all", data="gmm", d=3, n_ref=1_000_000,
             n_query=1_000_000, k=10, leaf=32, precision="fp32"),
        # tabular features with a few crowded clusters
        dict(name="pair_2m_d8_k10", op="all", data="zipf", d=8, n_ref=2_000_000,
             n_query=2_000_000, k=10, leaf=32, precision="fp32"),
        # a neighbour graph of medium-dimensional descriptors, ragged size,
        # dimension between the strides, a list length between the sizes
        dict(name="self_150k_d13_k7", op="all", data="tanh", d=13, n_ref=150_001, n_query=0, k=7,
             leaf=32, precision="fp32"),
        # large descriptor base, matrix-core tiles
        dict(name="pair_4m_d16_k10_bf16", op="all", data="tanh", d=16, n_ref=4_000_000,
             n_query=1_000_000, k=10, leaf=32, precision="bf16"),
        # embedding retrieval with long lists, matrix-core tiles
        dict(name="pair_1m_d64_k50_bf16", op="all", data="linear", d=64, n_ref=1_000_000,
             n_query=262_144, k=50, leaf=32, precision="bf16"),
        # the same kind of retrieval in FP32, on trees the program keeps
        dict(name="search_100k_d64_k50", op="search", data="linear", d=64, n_ref=100_003,
             n_query=20_011, k=50, leaf=32, precision="fp32"),
        # the other instances of the meta-algorithm, on trees the program
        # keeps: farthest points (diameters, outliers) ...
        dict(name="furthest_1m_d3_k10", op="furthest", data="gmm", d=3, n_ref=1_000_000,
             n_query=1_000_000, k=10, leaf=32),
        # ... fixed-radius neighbourhoods (simulation, clustering) ...
        dict(name="range_1m_d3", op="range", data="gmm", d=3, n_ref=1_000_000, n_query=1_000_000,
             hi=0.2, leaf=32),
        # ... densities ...
        dict(name="kde_1m_d3", op="kde", data="gmm", d=3, n_ref=1_000_000, n_query=1_000_000,
             h=1.0, eps=1.0, leaf=32),
        # ... and the spanning tree of a new cloud (tree build included)
        dict(name="emst_1m_d3", op="emst", data="gmm", d=3, n_ref=1_000_000, n_query=0, leaf=32),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["points", "all", "all", "all", "all", "search", "search", "furthest", "range",
                     "kde", "emst"])
    leaf = rng.choice([16, 20, 32, 32, 32])
    if op == "points":
        d = rng.choice([2, 3, 3, 5, 8])
        return dict(op=op, data="gmm", d=d, n_ref=_log_int(rng, 10_000, 1_000_000),
                    n_query=_log_int(rng, 1, 5_000), k=rng.randint(1, 16), leaf=leaf,
                    precision="fp32")
    if op in ("all", "search"):
        d = rng.choice([2, 3, 3, 4, 6, 8, 10, 16, 16, 24, 32, 48, 64])
        data = (rng.choice(["uniform", "gmm"]) if d <= 4 else rng.choice(["gmm", "zipf"])
                if d <= 8 else "tanh" if d <= 16 else "linear")
        top = 1_500_000 if d <= 4 else 800_000 if d <= 8 else 600_000 if d <= 16 else 150_000
        precision = rng.choice(["fp32", "bf16"]) if d >= 9 else "fp32"
        n_ref = _log_int(rng, 3_000, top)
        own = rng.random() < 0.3 and d <= 16
        n_query = 0 if own else _log_int(rng, 1_000, top if d <= 16 else 40_000)
        k = rng.choice([1, 3, 5, 8, 10, 10, 15, 20]) if d <= 16 else rng.choice([5, 10, 25, 50])
        return dict(op=op, data=data, d=d, n_ref=n_ref, n_query=n_query, k=k, leaf=leaf,
                    precision=precision)
    if op == "furthest":
        return dict(op=op, data="gmm", d=rng.choice([2, 3, 5]), n_ref=_log_int(rng, 5_000, 1_000_000),
                    n_query=_log_int(rng, 5_000, 1_000_000), k=rng.randint(1, 20), leaf=leaf)
    if op == "range":
        n_ref = _log_int(rng, 5_000, 1_000_000)
        return dict(op=op, data="gmm", d=3, n_ref=n_ref, n_query=_log_int(rng, 5_000, 1_000_000),
                    hi=round(rng.uniform(0.1, 0.25) * (1e6 / n_ref) ** (1 / 3), 4), leaf=leaf)
    if op == "kde":
        return dict(op=op, data="gmm", d=rng.choice([2, 3]), n_ref=_log_int(rng, 5_000, 400_000),
                    n_query=_log_int(rng, 5_000, 1_000_000), h=round(rng.uniform(0.5, 1.5), 3),
                    eps=1.0, leaf=leaf)
    return dict(op="emst", data="gmm", d=rng.choice([2, 3, 3, 5]), n_ref=_log_int(rng, 5_000, 600_000),
                n_query=0, leaf=leaf)


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _mixture(g, n_sets, d, zipf):
    comps = 64 if zipf else 32
    means = torch.rand(comps, d, generator=g, device=DEV, dtype=torch.float64) * 100.0
    sig = torch.exp(torch.rand(comps, generator=g, device=DEV, dtype=torch.float64)
                    * math.log(10.0) + math.log(0.5))
    w = torch.ones(comps, device=DEV, dtype=torch.float64)
    if zipf:
        w = torch.arange(1, comps + 1, device=DEV, dtype=torch.float64) ** -1.2
    cdf = torch.cumsum(w / w.sum(), 0)
    out = []
    for n in n_sets:
        u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
        c = torch.searchsorted(cdf, u).clamp_(max=comps - 1)
        z = torch.randn(n, d, generator=g, device=DEV, dtype=torch.float64)
        out.append((means[c] + sig[c, None] * z).float().contiguous())
    return out


def _manifold(g, n_sets, d, tanh):
    latent, noise = (4, 0.01) if tanh else (10, 0.02)
    a = torch.randn(latent, d, generator=g, device=DEV, dtype=torch.float64)
    out = []
    for n in n_sets:
        x = torch.rand(n, latent, generator=g, device=DEV, dtype=torch.float64) @ a
        if tanh:
            x = torch.tanh(x)
        x += noise * torch.randn(n, d, generator=g, device=DEV, dtype=torch.float64)
        out.append(x.float().contiguous())
    return out


def _points(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    d, kind = case["d"], case["data"]
    sizes = [case["n_ref"]] + ([case["n_query"]] if case["n_query"] else [])
    if kind == "uniform":
        sets = [torch.rand(n, d, generator=g, device=DEV, dtype=torch.float64).float().contiguous()
                for n in sizes]
    elif kind in ("gmm", "zipf"):
        sets = _mixture(g, sizes, d, kind == "zipf")
    else:
        sets = _manifold(g, sizes, d, kind == "tanh")
    return sets[0], (sets[1] if len(sets) > 1 else None)


def prepare(case, seed):
    ref, query = _points(case, seed)
    state = dict(case=case, ref=ref, query=query)
    op = case["op"]
    if op == "points":
        state["rt"] = knn.knn_build_tree(ref, case["leaf"])
    elif op in ("search", "furthest", "range", "kde"):
        if query is not None:
            state["rt"], state["qt"] = knn.knn_build_tree_pair(ref, query, case["leaf"])
        else:
            state["rt"], state["qt"] = knn.knn_build_tree(ref, case["leaf"]), None
    if op == "range":
        # a simulation keeps its neighbour lists in buffers of one capacity
        # (twice the neighbours these sets have on average)
        room = int(2 * _neighbours(case) * case["n_query"]) + 4096
        state["idx"] = torch.zeros(room, dtype=torch.int64, device=DEV)
        state["dist"] = torch.zeros(room, dtype=torch.float32, device=DEV)
    return state


def _neighbours(case):
    """Mean number of references within hi of a query: about 30 at the listed
    density, proportional to the number of references and the volume."""
    return 30.0 * (case["hi"] / 0.2) ** 3 * case["n_ref"] / 1e6


def run(state):
    c = state["case"]
    op = c["op"]
    if op == "all":
        idx, dist, _ = knn.knn_all_knn(state["ref"], state["query"], c["k"], c["leaf"],
                                       precision=c["precision"],
                                       exclude_self=state["query"] is None)
        return {"idx": idx, "dist": dist}
    if op == "points":
        idx, dist, _ = knn.knn_search_points(state["rt"], state["query"], c["k"],
                                             precision=c["precision"])
        return {"idx": idx, "dist": dist}
    if op == "search":
        idx, dist, _ = knn.knn_search(state["rt"], state["qt"], c["k"], precision=c["precision"],
                                      exclude_self=state["qt"] is None)
        return {"idx": idx, "dist": dist}
    if op == "furthest":
        idx, dist, _ = knn.knn_search_furthest(state["rt"], state["qt"], c["k"])
        return {"idx": idx, "dist": dist}
    if op == "range":
        offsets, idx, dist, _ = knn.knn_range_search(state["rt"], state["qt"], 0.0, c["hi"])
        n = min(idx.numel(), state["idx"].numel())
        state["idx"][:n].copy_(idx[:n])
        state["dist"][:n].copy_(dist[:n])
        return {"offsets": offsets, "idx": state["idx"], "dist": state["dist"]}
    if op == "kde":
        f, _ = knn.knn_kde(state["rt"], state["qt"], c["h"], c["eps"])
        return {"f": f}
    tree = knn.knn_build_tree(state["ref"], c["leaf"])
    u, v, w, rounds, _ = knn.knn_emst(tree)
    tree.close()
    return {"u": u, "v": v, "w": w, "rounds": rounds}


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def work(case):
    """Points read once, results written once; operations: building a tree
    compares every point once per level, and every query evaluates at least
    the distances it returns (3d - 1 operations each)."""
    d, nr = case["d"], case["n_ref"]
    nq = case["n_query"] or nr
    op = case["op"]
    pair = 3 * d - 1

    def levels(n):
        return max(1.0, math.log2(max(2.0, n / case["leaf"])))

    read = 4 * d * (nr + (case["n_query"] or 0))
    build_r, build_q = nr * levels(nr), (case["n_query"] or 0) * levels(max(1, case["n_query"]))
    if op == "all":
        return dict(bytes=read + 12 * nq * case["k"], flops=nq * case["k"] * pair + build_r + build_q)
    if op == "points":
        # a prebuilt tree: each query reads one path of boxes and its results
        return dict(bytes=4 * d * nq + 12 * nq * case["k"] + nq * 8 * d * levels(nr),
                    flops=nq * case["k"] * pair + build_q)
    if op in ("search", "furthest"):
        return dict(bytes=read + 12 * nq * case["k"], flops=nq * case["k"] * pair)
    if op == "range":
        near = _neighbours(case)
        return dict(bytes=read + 8 * nq + 12 * nq * near, flops=nq * near * pair)
    if op == "kde":
        return dict(bytes=read + 8 * nq, flops=nq * case["leaf"] * (3 * d + 1))
    return dict(bytes=read + 20 * nr, flops=nr * pair + build_r)


# --------------------------------------------------------------------------
# the FP64 answer by brute force
# --------------------------------------------------------------------------
_MOST_PAIRS = 6e10  # brute force beyond this takes too long


def _blocks(case, q, r):
    """Squared distances (FP64, coordinate differences) in blocks of rows."""
    rows = max(1, int(1.5e8 // max(1, r.shape[0])))
    rt = r.double().t().contiguous()
    qd = q.double()
    for i in range(0, q.shape[0], rows):
        s = torch.zeros(min(rows, q.shape[0] - i), r.shape[0], dtype=torch.float64, device=DEV)
        for j in range(case["d"]):
            t = qd[i:i + rows, j, None] - rt[j][None, :]
            s.addcmul_(t, t)
        yield i, s


def exact(case, seed):
    op = case["op"]
    nq = case["n_query"] or case["n_ref"]
    if op in ("emst", "range") or nq * case["n_ref"] * max(1, case["d"] / 8) > _MOST_PAIRS:
        return None  # lists in traversal order have no order to compare by
    ref, query = _points(case, seed)
    q = ref if query is None else query
    if op == "kde":
        f = torch.empty(nq, dtype=torch.float64, device=DEV)
        for i, s in _blocks(case, q, ref):
            f[i:i + s.shape[0]] = torch.exp(s * (-0.5 / case["h"] ** 2)).sum(1)
        return {"f": f}
    k, own = case["k"], query is None and op != "furthest"
    dist = torch.empty(nq, k, dtype=torch.float64, device=DEV)
    for i, s in _blocks(case, q, ref):
        if own:
            n = s.shape[0]
            at = torch.arange(n, device=DEV)
            s[at, at + i] = float("inf")
        v = torch.topk(s, k, dim=1, largest=op == "furthest", sorted=True).values
        dist[i:i + s.shape[0]] = torch.sqrt(v)
    return {"idx": None, "dist": dist}
