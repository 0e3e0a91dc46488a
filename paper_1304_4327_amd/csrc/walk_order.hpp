// The order in which the depth-first k-NN walk (search_valu.hpp) meets two
// reference points.  That walk keeps, among equal distances at the k-th
// place, what it meets first; the kernels that visit the reference tree in
// another order settle such a tie by this rule, so a call returns the same
// neighbours whichever kernel serves it.  It runs only where two distances
// are equal to the last bit.
#pragma once

#include "search_valu.hpp"

namespace knnx {

// the leaf node (and its first position) that holds tree position pos of a tree over n points (a
// node's left child takes floor(c / 2) of its c points)
__device__ inline int leaf_node_of(int pos, int n, int first_leaf, int &start) {
    int node = 0, cnt = n;
    start = 0;
    while (node < first_leaf) {
        const int half = cnt >> 1;
        if (pos < start + half) {
            node = 2 * node + 1;
            cnt = half;
        } else {
            node = 2 * node + 2;
            start += half;
            cnt -= half;
        }
    }
    return node;
}

// Whether the walk of the slot of query leaf qleaf (1 << ng_log2 sibling
// leaves) meets tree position pb before pa: of the two children of their
// lowest common ancestor, the one nearer to the slot's union box is entered
// first (the left one on equal keys); within a leaf the smaller position, for
// a BF16 request (a.walk_ties 0) the rows of the query's half of the tile
// first.
// The keys are computed as the walk computes them.  Wave-uniform arguments,
// every lane active.
template <int D>
__device__ inline bool walk_meets_second_first(const SearchArgs &a, int pa, int pb, int qleaf,
                                               int ng_log2) {
    constexpr int DP = stride_for(D);
    constexpr float kInf = __builtin_inff();
    const int lane = threadIdx.x & 63;
    const int n = a.rrange[0].y;
    int sa, sb;
    int na = leaf_node_of(pa, n, a.r_first_leaf, sa), nb = leaf_node_of(pb, n, a.r_first_leaf, sb);
    if (na == nb) {
        const int ha = ((pa - sa) >> 2) & 1, hb = ((pb - sb) >> 2) & 1;
        if (!a.walk_ties && ha != hb) return hb == (qleaf & 1);
        return pb < pa;
    }
    while (((na - 1) >> 1) != ((nb - 1) >> 1)) {
        na = (na - 1) >> 1;
        nb = (nb - 1) >> 1;
    }
    const int l0 = (qleaf >> ng_log2) << ng_log2;
    const int l1 = min(l0 + (1 << ng_log2), a.q_n_leaves);
    auto key = [&](int node) {
        const float *b = a.rbox + int64_t(node) * 2 * DP;
        float u = 0.f;
        auto gap = [&](int j) {
            float lo = kInf, hi = -kInf;
            for (int l = l0; l < l1; ++l) {
                const float *qb = a.qbox + int64_t(a.q_first_leaf + l) * 2 * DP;
                lo = fminf(lo, qb[j]);
                hi = fmaxf(hi, qb[DP + j]);
            }
            return fmaxf(fmaxf(b[j] - hi, lo - b[DP + j]), 0.0f);
        };
        if constexpr (D >= 16) {
            const float ug = lane < DP ? gap(lane < DP ? lane : 0) : 0.f;
            u = sum_dim_lanes<DP>(ug * ug);
        } else {
            for (int j = 0; j < D; ++j) {
                const float ug = gap(j);
                u = fmaf(ug, ug, u);
            }
        }
        return uniform_f(u);
    };
    const int left = min(na, nb), right = max(na, nb);
    const bool right_first = key(right) < key(left);
    return right_first ? nb == right : nb == left;
}

}  // namespace knnx
