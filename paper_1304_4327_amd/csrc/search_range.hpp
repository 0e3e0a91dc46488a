// Range-search kernel (Section "Range Search", Algorithms 5 and 6): for every
// query point every reference point at a distance in [lo, hi].
//
// Mapping as in the k-NN kernel: a wavefront owns 64 / 2^LG consecutive
// query leaves (lane = query point) and walks the reference tree
// (tree_walk).  Score treats each query point as a singleton node: the lane
// keeps a reference node unless its box lies entirely nearer than lo or
// entirely farther than hi (d_max < lo or d_min > hi; the printed test on
// d_min alone would drop overlapping nodes whose farther points are in
// range), with a 2^-16 relative slack for FP32 rounding.  BaseCase filters
// with FP32 squared distances (a relative slack covers their rounding) and
// decides every surviving pair exactly in FP64: lo^2 <= s <= hi^2, with s the
// FP64 squared distance of the FP32 inputs (products rounded, summed in
// dimension order) and lo^2, hi^2 squared in FP64 -- the same decision, bit
// for bit, as a plain FP64 loop over the dimensions.
//
// Two passes over the same traversal: the count pass writes each query's
// number of neighbours (original row order); after an exclusive scan of the
// counts the fill pass writes each query's neighbours from its offset on,
// in the order the traversal meets them (the paper's lists are unordered).
#pragma once

#include "walk.hpp"

namespace knnx {

struct RangeArgs {
    const float *rpts, *rbox, *rlpts;
    const int32_t *rperm;
    const int2 *rrange;
    int r_leaf_slots, r_first_leaf;
    const float *qpts, *qbox;
    const int32_t *qperm;
    const int2 *qrange;
    int q_first_leaf, q_n_leaves;
    double lo2, hi2;      // exact decision
    float s_lo, s_hi;     // Score thresholds on squared distances (with slack)
    // BaseCase FP32 filter: a pair outside [t_lo, t_hi) is out of range, one
    // inside [in_lo, in_hi] in range; FP64 decides between them
    // (in_lo == 0: no lower limit; wide: FP32 may overflow, FP64 decides all)
    float t_lo, t_hi, in_lo, in_hi;
    int wide;
    int prune, self;
    int split;               // waves per slot of query leaves (split_for)
    int64_t *counts;         // count pass: per original query row
    const int64_t *offsets;  // fill pass: exclusive prefix sums of the counts
    int64_t *out_idx;
    float *out_dist;
    unsigned long long *stats;  // ST_SCORE, ST_TILES, ST_PAIRS, ST_INSERTS (results)
};

template <int DP, int LG, bool FILL>
__global__ __launch_bounds__(256) void k_range(const RangeArgs a) {
    constexpr int NG = 64 >> LG;
    const int lane = threadIdx.x & 63;
    const int raw = uniform_i(xcd_remap(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6));
    const int wave = raw >> a.split, part = raw & ((1 << a.split) - 1);
    if (wave * NG >= a.q_n_leaves) return;
    const int g = lane >> LG, li = lane & ((1 << LG) - 1);
    const int slot = wave * NG + g;
    const bool has_leaf = slot < a.q_n_leaves;
    const int2 qr = has_leaf ? a.qrange[a.q_first_leaf + slot] : make_int2(0, 0);
    const bool point = has_leaf && li < qr.y;
    const bool valid = point && in_part<LG>(lane, part, a.split);
    if (!ballot(valid)) return;
    const int qpos = qr.x + li;
    // every lane keeps its point, also the ones of other parts: the visit
    // order follows lane 0's, so each query's list keeps its order
    float q[DP];
    {
        const float *qp = a.qpts + int64_t(point ? qpos : 0) * DP;
#pragma unroll
        for (int j = 0; j < DP; ++j) q[j] = point ? qp[j] : 0.f;
    }
    const int64_t row = valid ? int64_t(a.qperm[qpos]) : 0;
    int64_t out = 0;
    if constexpr (FILL) out = valid ? a.offsets[row] : 0;
    int found = 0;
    uint32_t n_score = 0, n_tiles = 0;
    uint64_t n_pairs = 0;
    const int n_valid = __popcll(ballot(valid));

    auto score = [&](int node, float &key) -> bool {
        ++n_score;
        float dmin2, dmax2;
        box_dist2<DP>(q, a.rbox + int64_t(node) * 2 * DP, dmin2, dmax2);
        // order key: the first lane's nearest distance (lane 0 is a point of
        // the wave's first leaf)
        key = uniform_f(dmin2);
        const bool keep = valid && (!a.prune || (!(dmin2 > a.s_hi) && !(dmax2 < a.s_lo)));
        return ballot(keep) != 0;
    };
    // (slots of a leaf are a multiple of 8: whole batches stay inside it)
    constexpr int CH = DP >= 32 ? 1 : 32 / DP;
    auto leaf = [&](int node) {
        ++n_tiles;
        const int2 rr = a.rrange[node];
        const int base = uniform_i(rr.x);
        const int cnt = uniform_i(rr.y);
        const float *rp = a.rlpts + int64_t(node - a.r_first_leaf) * a.r_leaf_slots * DP;
        n_pairs += uint64_t(cnt) * uint64_t(n_valid);
        // 32 slots at a time into one bit per pair (the sign of the squared
        // distance minus a threshold, shifted in), then one survivor per lane
        // and round: a leaf costs as many rounds as its busiest lane has
        // survivors, not one for every slot that some lane keeps (1M x 1M, d =
        // 3, r = 0.2: 77 hits a leaf and wave over 32 slots).  The count pass
        // adds the pairs that are in range beyond rounding and decides only
        // the others in FP64.
        for (int r0 = 0; r0 < cnt; r0 += 32) {
            const int r1 = min(cnt, r0 + 32);
            uint32_t hi = 0, lo = 0, in_hi = 0, in_lo = 0;  // bit k: the k-th slot from the end
            for (int t0 = r0; t0 < r1; t0 += CH) {
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    float sd = 0.f;
#pragma unroll
                    for (int j = 0; j < DP; ++j) {
                        const float df = q[j] - rp[(t0 + c) * DP + j];
                        sd = fmaf(df, df, sd);
                    }
                    auto shift_in = [](uint32_t m, float v) {
                        return __builtin_amdgcn_alignbit(m, __float_as_uint(v), 31);
                    };
                    hi = shift_in(hi, sd - a.t_hi);
                    if constexpr (!FILL) in_hi = shift_in(in_hi, sd - a.in_hi);
                    if (a.in_lo > 0.f) {  // uniform
                        lo = shift_in(lo, sd - a.t_lo);
                        if constexpr (!FILL) in_lo = shift_in(in_lo, sd - a.in_lo);
                    }
                }
            }
            // bit k: slot r0 + k (batches may reach past r1: those bits go)
            const int done = (r1 - r0 + CH - 1) / CH * CH;
            auto align = [&](uint32_t m) { return __brev(m) >> (32 - done); };
            const uint32_t rows = r1 - r0 >= 32 ? ~0u : (1u << (r1 - r0)) - 1u;
            uint32_t m = !valid ? 0u : a.wide ? rows : align(hi & ~lo) & rows;
            if (a.self && qpos - base - r0 >= 0 && qpos - base - r0 < 32) m &= ~(1u << (qpos - base - r0));
            if constexpr (!FILL) {
                const uint32_t sure = a.wide ? 0u : m & align(in_hi & ~in_lo);
                found += __popc(sure);
                m &= ~sure;
            }
            while (ballot(m != 0)) {
                const bool has = m != 0;
                const int t = r0 + (has ? __builtin_ctz(m) : 0);
                m &= m - 1u;
                const double x = d2_fp64_unfused<DP>(q, rp + t * DP);
                if (has && x >= a.lo2 && x <= a.hi2) {
                    if constexpr (FILL) {
                        a.out_idx[out + found] = a.rperm[base + t];
                        a.out_dist[out + found] = (float)sqrt(x);
                    }
                    ++found;
                }
            }
        }
    };
    tree_walk(a.r_first_leaf, score, leaf, [](float k0, float k1) { return k1 < k0; });

    if constexpr (!FILL) {
        if (valid) a.counts[row] = found;
    }
    if (a.stats) {
        int f = found;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) f += __shfl_xor(f, off);
        if (lane == 0) {
            atomicAdd(&a.stats[ST_SCORE], (unsigned long long)n_score);
            atomicAdd(&a.stats[ST_TILES], (unsigned long long)n_tiles);
            atomicAdd(&a.stats[ST_PAIRS], (unsigned long long)n_pairs);
            atomicAdd(&a.stats[ST_INSERTS], (unsigned long long)f);
        }
    }
}

template <int DP>
hipError_t launch_range(const RangeArgs &a, int lg, bool fill, int grid, hipStream_t s) {
    if (lg == 5) {
        if (fill)
            k_range<DP, 5, true><<<grid, 256, 0, s>>>(a);
        else
            k_range<DP, 5, false><<<grid, 256, 0, s>>>(a);
    } else {
        if (fill)
            k_range<DP, 6, true><<<grid, 256, 0, s>>>(a);
        else
            k_range<DP, 6, false><<<grid, 256, 0, s>>>(a);
    }
    return hipGetLastError();
}

}  // namespace knnx
