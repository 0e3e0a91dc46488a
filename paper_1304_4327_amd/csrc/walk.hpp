// The pruning dual-tree traversal's reference-side walk (Algorithm 1 with a
// query node fixed per wavefront), shared by the range-search, kernel
// density and Boruvka kernels: a depth-first walk over the heap-ordered
// reference tree without a stack.  One bit per depth records which child
// was entered first; when the walk climbs back to that child, the other one
// is scored (bounds only change monotonically, so the late score can only
// prune more).  Every (query node, reference node) pair is scored at most
// once, and a pruned node's subtree is never entered.
//
// score(node, key) -> bool : Score() of a reference node, wave-uniform;
//                            key is a wave-uniform order key
// leaf(node)               : BaseCase() over a kept reference leaf
// right_first(k0, k1)      : whether to enter the right child first when
//                            both are kept
// The leaf call sits in the outer loop and the walk in the inner one, so the
// state leaf() updates is not carried through the walk's loop.
#pragma once

#include "search_valu.hpp"

namespace knnx {

template <class Score, class Leaf, class Order>
__device__ __forceinline__ void tree_walk(int first_leaf, Score &&score, Leaf &&leaf,
                                          Order &&right_first) {
    float m0, m1;
    int node = 0, depth = 0;
    uint64_t firstbits = 0;
    bool down = score(0, m0);
    if (!down) return;
    for (;;) {
        bool at_leaf = false;
        for (;;) {
            if (down) {
                if (node >= first_leaf) {
                    at_leaf = true;
                    break;
                }
                const int c0 = 2 * node + 1, c1 = c0 + 1;
                const bool k0 = score(c0, m0);
                const bool k1 = score(c1, m1);
                if (!k0 && !k1) {
                    down = false;
                    continue;
                }
                const bool right = k1 && (!k0 || right_first(m0, m1));
                if (right)
                    firstbits |= (uint64_t(1) << depth);
                else
                    firstbits &= ~(uint64_t(1) << depth);
                node = uniform_i(right ? c1 : c0);
                ++depth;
            } else {
                if (node == 0) break;
                --depth;
                const bool is_right = (node & 1) == 0;
                const bool first_right = (firstbits >> depth) & 1;
                if (is_right == first_right) {
                    const int other = is_right ? node - 1 : node + 1;
                    if (score(other, m0)) {
                        node = other;
                        ++depth;
                        down = true;
                        continue;
                    }
                }
                node = uniform_i((node - 1) >> 1);
            }
        }
        if (!at_leaf) break;
        leaf(node);
        down = false;
    }
}

// The same walk for a Score that depends on the two boxes alone: five levels
// below a node are scored at once, a node per lane, and the walk below it is
// bit arithmetic on the ballots.  Lane v holds the descendant with heap index
// v under the block's root (v = 1), which is node (root << level) + v - 1.
// The second children still to be visited are bits of a mask; they are
// siblings of the path's nodes, one a level, so the next one is the highest.
// The first block takes the levels that are left over, so the last one is
// full.  Nodes, and the two children of each, are visited in tree_walk's
// order.
//
// score(node, on, keep, appr, key) : per lane, node of that lane (on: exists)
// appr(node)    : wave-uniform, a visited node's approximation
// leaf(node)    : wave-uniform, BaseCase
// returns the number of nodes that the walk looked at
template <class Score, class Appr, class Leaf>
__device__ __forceinline__ uint32_t tree_walk_blocks(int first_leaf, Score &&score, Appr &&appr,
                                                     Leaf &&leaf) {
    constexpr int kLevels = 5;
    const int lane = threadIdx.x & 63;
    const int lane_level = 31 - __clz(lane | 1);
    const int height = 31 - __clz(first_leaf + 1);
    uint64_t keep = 0, ap = 0, right = 0, todo = 0;
    auto block = [&](int root, int levels) {
        const bool on = lane >= 1 && lane_level <= levels;
        const int node = on ? (root << lane_level) + lane - 1 : 0;
        bool k, p;
        float key;
        score(node, on, k, p, key);
        keep = ballot(k);
        ap = ballot(p);
        // at the left child's bit: the right one is nearer
        right = ballot(dpp_f<0xB1>(key) < key);
    };
    uint32_t n = 1;
    int root = 0, levels = height % kLevels ? height % kLevels : min(height, kLevels);
    block(0, levels);
    if (ap & 2) appr(0);
    if (!(keep & 2)) return n;
    // the blocks above the current one, one a lane
    int sp = 0, s_root = 0;
    uint64_t s_keep = 0, s_ap = 0, s_right = 0, s_todo = 0;
    int v = 1;
    for (;;) {
        int node;
        bool at_leaf = false;
        for (;;) {
            const int level = 31 - __builtin_clz(v);
            node = (root << level) + v - 1;
            if (node >= first_leaf) {
                at_leaf = true;
                break;
            }
            if (level == levels) {
                const bool here = lane == sp;
                s_root = here ? root : s_root;
                s_keep = here ? keep : s_keep;
                s_ap = here ? ap : s_ap;
                s_right = here ? right : s_right;
                s_todo = here ? todo : s_todo;
                ++sp;
                root = node;
                levels = kLevels;
                todo = 0;
                v = 1;
                block(root, kLevels);
            }
            n += 2;
            const int c0 = 2 * v;
            const int a2 = int(ap >> c0) & 3, k2 = int(keep >> c0) & 3;
            if (a2) {
                if (a2 & 1) appr(2 * node + 1);
                if (a2 & 2) appr(2 * node + 2);
            }
            if (k2 == 3) {
                const int r = int(right >> c0) & 1;
                v = c0 + r;
                todo |= uint64_t(1) << (c0 + 1 - r);
            } else if (k2) {
                v = c0 + (k2 >> 1);
            } else {
                break;
            }
        }
        if (at_leaf) leaf(node);
        while (todo == 0) {
            if (sp == 0) return n;
            --sp;
            auto get = [&](uint64_t x) {
                return uint64_t(uint32_t(__builtin_amdgcn_readlane(int(x), sp))) |
                       uint64_t(uint32_t(__builtin_amdgcn_readlane(int(x >> 32), sp))) << 32;
            };
            root = __builtin_amdgcn_readlane(s_root, sp);
            keep = get(s_keep);
            ap = get(s_ap);
            right = get(s_right);
            todo = get(s_todo);
            if (sp == 0) levels = height % kLevels ? height % kLevels : kLevels;
        }
        v = 63 - __builtin_clzll(todo);
        todo &= ~(uint64_t(1) << v);
    }
}

// squared distance from a point to a box: nearest (gap) and farthest point
template <int DP>
__device__ __forceinline__ void box_dist2(const float (&q)[DP], const float *b, float &dmin2,
                                          float &dmax2) {
    float lo2 = 0.f, hi2 = 0.f;
#pragma unroll
    for (int j = 0; j < DP; ++j) {
        const float lo = b[j], hi = b[DP + j];
        const float g = fmaxf(fmaxf(lo - q[j], q[j] - hi), 0.0f);
        const float f = fmaxf(fmaxf(q[j] - lo, hi - q[j]), 0.0f);
        lo2 = fmaf(g, g, lo2);
        hi2 = fmaf(f, f, hi2);
    }
    dmin2 = lo2;
    dmax2 = hi2;
}

// FP64 squared distance of FP32 coordinates with every product rounded
// (no fused multiply-add), summed in dimension order: bit for bit the value
// of a plain sequential FP64 loop, so a decision taken on it matches one
// taken by such a loop (padding dimensions add exact zeros)
template <int DP>
__device__ __forceinline__ double d2_fp64_unfused(const float (&q)[DP], const float *r) {
#pragma clang fp contract(off)
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < DP; ++j) {
        const double t = (double)q[j] - (double)r[j];
        s = s + t * t;
    }
    return s;
}

}  // namespace knnx
