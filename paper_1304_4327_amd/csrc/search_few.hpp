// k-NN of few query points (stride <= 16): one wavefront per query point.
//
// What bounds it.  A small query set leaves the chip nearly empty, and the
// walk that carries a slot of query leaves per wave (search_valu.hpp) then
// lasts as long as its slowest wave: a chain of dependent box loads, longer
// the more of the reference tree the slot's scattered queries open together.
// 257 new points against 100,000 in d = 3, k = 8, took 1.84 ms that way (8
// waves); one query per wave on the same walk still 0.6 ms (its chain is one
// box pair per step).  Here the wave's 64 lanes work on the reference side of
// one query: a step scores 64 nodes, six levels below the node it expands
// (their boxes are contiguous in heap order), and a tile is two leaves, a
// lane per point.  The dependent chain of a query is about a dozen steps.
//
// Traversal: Algorithm 1 with the query point as the query node {p} (lambda
// = 0, so B({p}) = D_p[k]); of an expanded node's descendants the nearest is
// entered first, until none is within the bound.  Every (p, node) pair is
// scored at most once.
//
// List: sorted across the lanes, lane t the t-th smallest distance; few new
// candidates are inserted one by one, many are sorted by a bitonic network
// and merged.  Distances are those of the walk (FP32 differences up to d = 8,
// above that FP64 of the FP32 points).  The lanes past the k-th entry keep
// what ties with it, and the choice among equal distances follows the walk's
// order, so both kernels return the same neighbours.
#pragma once

#include "walk_order.hpp"

namespace knnx {

// minimum over the wave (wave-uniform result), lane moves by DPP alone: rows
// of 16, then each row's last lane to the next row, then to the upper half
__device__ inline float wave_min(float v) {
    v = reduce16(v, OpMin());
    const int a = __builtin_bit_cast(int, v);
    v = fminf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(a, a, 0x142, 0xA, 0xF, false)));
    const int b = __builtin_bit_cast(int, v);
    v = fminf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(b, b, 0x143, 0xC, 0xF, false)));
    return __int_as_float(__builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
// lane l's value from lane l - 1; lane 0 gets `first`
__device__ inline int lane_before(int v, int first) {
    return __builtin_amdgcn_update_dpp(first, v, 0x138, 0xF, 0xF, false);
}

template <int D>
__global__ __launch_bounds__(256) void k_search_few(const SearchArgs a) {
    constexpr int DP = stride_for(D);
    constexpr bool RESCORE = D > 8;
    constexpr float kInf = __builtin_inff();
    constexpr float kSlack = 1.0f + 0x1p-16f;            // prune slack (squared)
    constexpr float kGamma = 1.0f + (D + 6) * 0x1p-24f;  // FP32 filter slack
    const int lane = threadIdx.x & 63;
    const int n_q = a.qrange[0].y;
    const int qpos = uniform_i(xcd_remap(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6));
    if (qpos >= n_q) return;
    float q[D];
#pragma unroll
    for (int j = 0; j < D; ++j) q[j] = a.qpts[int64_t(qpos) * DP + j];
    const int kk = a.k + (a.self ? 1 : 0);  // list length (self match included)

    float x = kInf;  // the list: lane t holds the t-th entry
    int id = -1;
    float kth = kInf;  // entry kk - 1; what equals it is kept behind it
    auto at = [&](float v, int l) {
        return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
    };
    // compare-exchange with lane ^ m on (distance, position)
    auto exchange = [&](float &v, int &p, int m, bool up) {
        const float ov = __shfl_xor(v, m);
        const int op = __shfl_xor(p, m);
        const bool other_less = ov < v || (ov == v && op < p);
        const bool low = (lane & m) == 0;
        if (up ? low == other_less : low != other_less) {
            v = ov;
            p = op;
        }
    };
    auto add = [&](float v, int p, bool cand) {
        uint64_t m = ballot(cand);
        if (!m) return;
        if (__popcll(m) <= 6) {
            while (m) {
                const int c = __builtin_ctzll(m);
                m &= m - 1;
                const float nv = at(v, c);
                if (!(nv <= kth)) continue;
                const int np = __builtin_amdgcn_readlane(p, c);
                // entries above the new one move up a lane
                const float xp = __int_as_float(lane_before(__float_as_int(x), 0xff800000));
                const int ip = lane_before(id, -1);
                const bool above = x > nv, shift = xp > nv;
                x = above ? (shift ? xp : nv) : x;
                id = above ? (shift ? ip : np) : id;
                kth = at(x, kk - 1);
            }
            return;
        }
        v = cand ? v : kInf;
        // (distinct positions: the exchanges agree in both lanes)
        p = cand ? p : 0x7fffff00 + lane;
        for (int size = 2; size <= 64; size <<= 1)
            for (int st = size >> 1; st > 0; st >>= 1) exchange(v, p, st, (lane & size) == 0);
        const float rv = __shfl(v, 63 - lane);
        const int rp = __shfl(p, 63 - lane);
        if (rv < x || (rv == x && rp < id && rv < kInf)) {
            x = rv;
            id = rp;
        }
        for (int st = 32; st > 0; st >>= 1) exchange(x, id, st, true);
        kth = at(x, kk - 1);
    };

    // one tile: leaf n0, and leaf n1 in the upper lanes (or none: n1 < 0)
    const bool two = a.r_leaf_slots <= 32;
    auto tile = [&](int n0, int n1) {
        const int node = two && lane >= 32 ? n1 : n0;
        const int s = two ? lane & 31 : lane;
        const int2 rr = a.rrange[max(node, 0)];
        const bool on = node >= 0 && s < rr.y;
        const float *rp =
            a.rlpts + (int64_t(max(node, a.r_first_leaf) - a.r_first_leaf) * a.r_leaf_slots + (on ? s : 0)) * DP;
        float r[DP];
#pragma unroll
        for (int j = 0; j < DP; j += 4) {
            const float4 t = *reinterpret_cast<const float4 *>(rp + j);
            r[j] = t.x;
            r[j + 1] = t.y;
            r[j + 2] = t.z;
            r[j + 3] = t.w;
        }
        float v = 0.f;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const float df = q[j] - r[j];
            v = fmaf(df, df, v);
        }
        bool cand = on && v <= (RESCORE ? kth * kGamma : kth) && v < kInf;
        if constexpr (RESCORE) {
            if (!ballot(cand)) return;
            v = (float)d2_fp64<D>(q, r);
            cand = cand && v <= kth && v < kInf;
        }
        add(v, rr.x + s, cand);
    };

    // nodes six levels at a time: the first step takes the remainder
    const int depth = 31 - __clz(a.r_first_leaf + 1);
    const int steps = (depth + 5) / 6;
    const int s0 = depth - 6 * (steps - 1);
    auto box_d2 = [&](int first, int n) -> float {
        float d = kInf;
        if (lane < n) {
            const float *b = a.rbox + int64_t(first + lane) * 2 * DP;
            d = 0.f;
            float lo[DP], hi[DP];
#pragma unroll
            for (int j = 0; j < DP; j += 4) {
                const float4 l = *reinterpret_cast<const float4 *>(b + j);
                const float4 h = *reinterpret_cast<const float4 *>(b + DP + j);
                lo[j] = l.x, lo[j + 1] = l.y, lo[j + 2] = l.z, lo[j + 3] = l.w;
                hi[j] = h.x, hi[j + 1] = h.y, hi[j + 2] = h.z, hi[j + 3] = h.w;
            }
#pragma unroll
            for (int j = 0; j < D; ++j) {
                const float gap = fmaxf(fmaxf(lo[j] - q[j], q[j] - hi[j]), 0.0f);
                d = fmaf(gap, gap, d);
            }
        }
        return d;
    };
    // the nearest unvisited node of a step's 64, or -1 when none is in reach
    auto pick = [&](float &d) -> int {
        const float m = wave_min(d);
        if (!(m < kInf) || m > kth * kSlack) return -1;
        const int l = __builtin_ctzll(ballot(d == m));
        if (lane == l) d = kInf;
        return l;
    };
    // depth first over the steps; the pending distances of the steps above
    // wait in LDS (each lane its own), and the node list of a step follows
    // from the node entered from it
    __shared__ float s_pending[4][5][64];
    float(*pending)[64] = s_pending[threadIdx.x >> 6];
    if (steps == 0) {
        tile(0, -1);
    } else {
        int t = 0, node = 0;  // the node expanded at step t
        int first = (1 << s0) - 1;
        float d = box_d2(first, 1 << s0);
        for (;;) {
            const int l = pick(d);
            if (l < 0) {
                if (t == 0) break;
                --t;
                const int s = t == 0 ? s0 : 6;
                first = (((node + 1) >> s) << s) - 1;
                node = ((node + 1) >> s) - 1;
                d = pending[t][lane];
            } else if (t == steps - 1) {
                const int l1 = two ? pick(d) : -1;
                tile(first + l, l1 < 0 ? -1 : first + l1);
            } else {
                pending[t][lane] = d;
                ++t;
                node = first + l;
                first = ((node + 1) << 6) - 1;
                d = box_d2(first, 64);
            }
        }
    }

    // ---- write-out -----------------------------------------------------------
    if (a.self) {  // the query's own point leaves the list
        const uint64_t own = ballot(id == qpos);
        if (own) {
            const int p = __builtin_ctzll(own);
            const float xn = __shfl_down(x, 1);
            const int in = __shfl_down(id, 1);
            if (lane >= p) {
                x = lane < 63 ? xn : kInf;
                id = lane < 63 ? in : -1;
            }
        }
    }
    const float xk = at(x, a.k - 1);
    if (xk < kInf && at(x, a.k) == xk) {
        // equal distances at the k-th place: the ones the walk meets first
        const uint64_t grp = ballot(x == xk);
        const int g0 = __builtin_ctzll(grp), g1 = 63 - __builtin_clzll(grp);
        int q0;
        const int ql = leaf_node_of(qpos, n_q, a.q_first_leaf, q0) - a.q_first_leaf;
        for (int e = g1; e > g0; --e) {
            bool swapped = false;
            for (int t = g0; t < e; ++t) {
                const int i0 = __builtin_amdgcn_readlane(id, t);
                const int i1 = __builtin_amdgcn_readlane(id, t + 1);
                if (walk_meets_second_first<D>(a, i0, i1, ql, 6 - a.lpl_log2)) {
                    if (lane == t) id = i1;
                    if (lane == t + 1) id = i0;
                    swapped = true;
                }
            }
            if (!swapped) break;
        }
    }
    const bool real = lane < a.k && x < kInf && id >= 0;
    const int p = real ? id : 0;
    float key = kInf;
    int o = 0x7fffffff - 63 + lane;
    if (real) {
        key = (float)sqrt(d2_fp64<D>(q, a.rpts + int64_t(p) * DP));
        o = a.rperm[p];
    }
    int rank = 0;
    for (int i = 0; i < a.k; ++i) {
        const float ki = at(key, i);
        const int oi = __builtin_amdgcn_readlane(o, i);
        rank += (ki < key) || (ki == key && oi < o);
    }
    if (lane < a.k) {
        const int64_t row = int64_t(a.qperm[qpos]) * a.k;
        a.out_idx[row + rank] = real ? o : -1;
        a.out_dist[row + rank] = key;
    }
}

template <int D>
hipError_t launch_search_few(const SearchArgs &a, int64_t n_q, hipStream_t s) {
    k_search_few<D><<<int((n_q + 3) / 4), 256, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace knnx
