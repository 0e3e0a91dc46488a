// High-dimensional k-NN (stride 64, and FP32 requests at stride 32): a sweep over blocks of reference leaves
// on the matrix unit, two query leaves per wavefront.  The traversal is the
// pruning dual-tree traversal of Algorithm 1 in another order: every
// (query node, reference leaf) pair is scored once and pruned when its
// d_min exceeds the bound.
//
// Why a sweep.  With d = 64 and tens of thousands of reference leaves the
// nearest-first walk enters most leaves anyway and costs a chain of dependent
// box loads; a sweep scores 32 leaves at once and loads the next kept leaf
// while the current one is processed.
//
// What bounds it: the operand rows of the kept leaves (4 KB each), which
// come from beyond L2 nearly every time.  With one query leaf per wave (and
// each query's list dealt over two lanes) the 1M x 262,144 points, d = 64,
// k = 50 search read 374 GB in 86.7 ms; with two leaves per wave each operand
// read serves 64 queries, a lane holds its query's whole list (so its k-th
// distance needs no merge of half-lists), and the operand layout makes every
// load instruction one contiguous 1 KB: 243 GB (and 11 GB of registers spilled)
// in 63 ms, 4 TB/s where a large copy reaches 5.1.  At stride 32 the FP32 search of
// 83,781 points by 34,155 queries (d = 32, k = 10) took 34.1 ms in the walk,
// 2.0 ms here.
//
// Reference side (k_wsweep_prep, once per search): every row as BF16
// -2 (r - C_B) centred on its block's centre C_B, the FP32 row norms, and
// each leaf's enclosing ball relative to C_B.
//
// Score.  Blocks of 32 consecutive reference leaves (one subtree), nearest
// first per workgroup.  A query p keeps leaf L unless the low end of
// |p - C_L|^2 (a BF16 tile and its proven margin) exceeds (b_p + rho_L)^2,
// b_p = sqrt(min(D_p[k], B(leaf of p))).  A wave multiplies the leaves that
// any of its 64 queries keeps.
//
// BaseCase.  The BF16 tile is a filter only: a row whose value minus the
// margin of bf16_tile.hpp cannot beat the bound is skipped, every other one
// gets its distance from the FP32 points in FP64, and only that value enters
// a list or a bound.  So the search is exact for either precision request.
// Where a block's norms or a query's distance to its centre lie outside the
// range that the margin covers (coordinates some 1e17 apart and more, or all
// within 1e-15), its leaves are scored by their boxes and its rows filtered by
// FP32 differences, as in the walk.
//
// Lists.  K >= kk + 2 slots (kk = k, or k + 1 with the query's own point):
// the k-th distance is slot K - 3, and the two extra entries hold what ties
// with it, so that the choice among equal distances does not depend on the
// order of the sweep: `walk_ties` (FP32 requests) keeps what the depth-first
// walk meets first, as that kernel does; else the smaller original index
// wins among equal output distances.
//
// Few query leaves (`parts`): the four waves of a workgroup share one pair of
// leaves, each taking every fourth block; they exchange their k-th distances
// through LDS and merge their lists at the end.
#pragma once

#include "search_mfma.hpp"
#include "walk_order.hpp"

namespace knnx {

constexpr int kPairSortMax = 2048;

template <int DP, int K>
struct PairLds {
    static constexpr int row = DP + 4;  // floats per query row (padded: a lane per row)
    // (at stride 32 the longest list of the parts form takes more)
    static constexpr size_t four_waves = size_t(4) * 64 * row * 4;
    static constexpr size_t one_list = size_t(64) * row * 4 + 64 * 4 + size_t(64) * K * 8;
    static constexpr size_t q_rows = four_waves > one_list ? four_waves : one_list;
    // the block order and its keys; while they are sorted (in the query rows'
    // space) the centre sits in the keys' space
    static constexpr size_t off_okey = q_rows;
    static constexpr size_t off_order = off_okey + size_t(kPairSortMax) * 4;
    static constexpr size_t bytes = off_order + size_t(kPairSortMax) * 2;
    // parts: rows of one pair, then the shared k-th distances, then one
    // wave's list
    static constexpr size_t off_kth = size_t(64) * row * 4;
    static constexpr size_t off_list = off_kth + 64 * 4;
    static_assert(off_list + size_t(64) * K * 8 <= q_rows, "one wave's list fits the query rows");
    static_assert(size_t(kPairSortMax) * 8 <= q_rows, "the sort fits the query rows");
};

template <int DP, int K>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(K <= 53 ? 2 : 1))) void
k_search_pair(const SearchArgs a) {
    using L = PairLds<DP, K>;
    constexpr int S = DP / 16;  // k-steps of 16 dimensions
    constexpr int E = DP / 8;
    constexpr int NB = kSweepBlock;
    constexpr float kInf = __builtin_inff();
    constexpr float kSlack = 1.0f + 0x1p-16f;
    __shared__ __align__(16) char smem[L::bytes];
    float *s_q = reinterpret_cast<float *>(smem);
    float *s_okey = reinterpret_cast<float *>(smem + L::off_okey);
    uint16_t *s_order = reinterpret_cast<uint16_t *>(smem + L::off_order);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = uniform_i(tid >> 6);
    const int jj = lane & 31, hh = lane >> 5;
    const bool parts = a.split != 0;
    const int n_list = a.q_n_leaves;
    const int wg_leaves = parts ? 2 : kPairLeaves;
    const int leaf0 = xcd_remap(blockIdx.x, gridDim.x) * wg_leaves;
    if (leaf0 >= n_list) return;  // whole workgroup
    auto leaf_on = [&](int sl) { return sl < n_list && (!a.active || a.active[sl] != 0); };
    bool any_leaf = false;
    for (int g = 0; g < wg_leaves; ++g) any_leaf |= leaf_on(leaf0 + g);
    if (!any_leaf) return;  // whole workgroup (fallback pass)

    const int slot = leaf0 + (parts ? 0 : 2 * w) + hh;  // this lane's query leaf
    const bool has_leaf = leaf_on(slot);
    const int qleaf = has_leaf ? slot : leaf0;
    const int qnode = a.q_first_leaf + qleaf;
    const int2 qr = has_leaf ? a.qrange[qnode] : make_int2(0, 0);
    const bool valid = jj < qr.y;
    const int qpos = qr.x + (valid ? jj : 0);
    const int n_valid = __popcll(ballot(valid));
    const int kk = a.k + (a.self ? 1 : 0);
    const int pad = K - kk - 2;  // unused front slots (they hold -inf)

    // union box centre of the workgroup's leaves (lane = dimension)
    float cl = 0.f;
    if (lane < DP) {
        float lo = kInf, hi = -kInf;
        for (int g = 0; g < wg_leaves; ++g) {
            if (leaf_on(leaf0 + g)) {
                const float *qb = a.qbox + int64_t(a.q_first_leaf + leaf0 + g) * 2 * DP;
                lo = fminf(lo, qb[lane]);
                hi = fmaxf(hi, qb[DP + lane]);
            }
        }
        cl = 0.5f * (lo + hi);
    }
    float *s_cen = s_okey;
    if (w == 0 && lane < DP) s_cen[lane] = cl;
    __syncthreads();

    const int nl = a.r_first_leaf + 1;  // reference leaves
    const int n_blocks = (nl + NB - 1) / NB;  // a power of two
    // Block order: up to kPairSortMax blocks nearest first by k_b = |c - C_b|
    // (1 - 2^-12) - lambda(b): d(q, r) >= k_b - R for every query within R of
    // c and every point of the block, so once k_b exceeds R plus a wave's
    // largest bound, no later block can hold a neighbour.  More blocks: outward
    // in tree order from the block the centre falls in, without an early end.
    const bool use_sort = n_blocks <= kPairSortMax;
    float R = 0.f;
    int sblock = 0;
    if (use_sort) {
        const int trow = tid >> 3, tcol = (tid & 7) * E;
        float tc[E];
#pragma unroll
        for (int e = 0; e < E; ++e) tc[e] = s_cen[tcol + e];
        // this query's |q - c|
        const float *qp = a.qpts + int64_t(qpos) * DP;
        float qn = 0.f;
#pragma unroll 4
        for (int u = 0; u < DP; u += 4) {
            const float4 x = *reinterpret_cast<const float4 *>(qp + u);
            const float4 c = *reinterpret_cast<const float4 *>(s_cen + u);
            const float g0 = x.x - c.x, g1 = x.y - c.y, g2 = x.z - c.z, g3 = x.w - c.w;
            qn = fmaf(g0, g0, fmaf(g1, g1, fmaf(g2, g2, fmaf(g3, g3, qn))));
        }
        R = uniform_f(reduce64(valid ? sqrtf(qn) : 0.f, OpMax())) * (1.0f + 0x1p-12f);
        uint64_t *s_sort = reinterpret_cast<uint64_t *>(smem);
        const int first = n_blocks - 1;  // heap index of block 0's node
        for (int b0 = 0; b0 < n_blocks; b0 += 32) {
            const int bi = b0 + trow;
            const bool vb = bi < n_blocks;
            const float *bx = a.rbox + int64_t(first + (vb ? bi : 0)) * 2 * DP;
            float sq = 0.f;
#pragma unroll
            for (int e = 0; e < E; e += 4) {
                const float4 lo = *reinterpret_cast<const float4 *>(bx + tcol + e);
                const float4 hi = *reinterpret_cast<const float4 *>(bx + DP + tcol + e);
                const float cv[4] = {0.5f * (lo.x + hi.x), 0.5f * (lo.y + hi.y), 0.5f * (lo.z + hi.z),
                                     0.5f * (lo.w + hi.w)};
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float df = cv[u] - tc[e + u];
                    sq = fmaf(df, df, sq);
                }
            }
            sq = reduce8(sq, OpAdd());
            if (vb && (tid & 7) == 0) {
                // (an overflow says nothing: such a block comes first)
                const float key =
                    sq < kInf ? sqrtf(sq) * (1.0f - 0x1p-12f) - a.rlam[first + bi] : -kInf;
                s_sort[bi] = (uint64_t(f2key(key)) << 32) | uint32_t(bi);
            }
        }
        // bitonic sort of the n_blocks (key, block) words, ascending
        for (int size = 2; size <= n_blocks; size <<= 1) {
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                __syncthreads();
                for (int i = tid; i < n_blocks / 2; i += 256) {
                    const int lo = 2 * stride * (i / stride) + (i & (stride - 1));
                    const int hi = lo + stride;
                    const uint64_t x = s_sort[lo], y = s_sort[hi];
                    if ((x > y) == ((lo & size) == 0)) {
                        s_sort[lo] = y;
                        s_sort[hi] = x;
                    }
                }
            }
        }
        __syncthreads();
        for (int i = tid; i < n_blocks; i += 256) {
            const uint64_t x = s_sort[i];
            s_order[i] = uint16_t(x & 0xffffu);
            s_okey[i] = key2f(uint32_t(x >> 32));
        }
        __syncthreads();
    } else {
        int node = 0;
        while (node < a.r_first_leaf) {
            const int c0 = 2 * node + 1;
            const float *b0 = a.rbox + int64_t(c0) * 2 * DP;
            const float *b1 = b0 + 2 * DP;
            const float g0 = lane < DP ? fmaxf(fmaxf(b0[lane] - cl, cl - b0[DP + lane]), 0.f) : 0.f;
            const float g1 = lane < DP ? fmaxf(fmaxf(b1[lane] - cl, cl - b1[DP + lane]), 0.f) : 0.f;
            const float d0 = uniform_f(reduce64(g0 * g0, OpAdd()));
            const float d1 = uniform_f(reduce64(g1 * g1, OpAdd()));
            node = uniform_i(d1 < d0 ? c0 + 1 : c0);
        }
        sblock = (node - a.r_first_leaf) / NB;
        __syncthreads();  // every wave has its centre; s_cen's space is free
    }
    const int n_steps = use_sort ? n_blocks : 2 * max(sblock, n_blocks - 1 - sblock) + 1;

    // the query rows (FP32): lane l's row, zero for idle lanes
    float *rows_w = s_q + (parts ? 0 : w * 64 * L::row);
    float *my_q = rows_w + lane * L::row;
    uint32_t *s_kth = reinterpret_cast<uint32_t *>(smem + L::off_kth);  // parts only
    if (!parts || w == 0) {
        for (int u = 0; u < DP; u += 4) {
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (valid) v = *reinterpret_cast<const float4 *>(a.qpts + int64_t(qpos) * DP + u);
            *reinterpret_cast<float4 *>(my_q + u) = v;
        }
        if (parts) s_kth[lane] = __float_as_uint(kInf);
    }
    __syncthreads();

    const float lam2 = has_leaf ? 2.0f * a.qlam[qnode] : 0.f;
    float lam2_anc = kInf;  // the pair's parent (when the tree has one)
    if (a.bound == KNN_BOUND_B && has_leaf && qnode > 0) lam2_anc = 2.0f * a.qlam[(qnode - 1) >> 1];
    const float seed = (a.seed && has_leaf) ? fmaxf(a.seed[qleaf], 0.0f) : kInf;
    const float seed2 = seed * seed;

    float dist[K];
    int idx[K];
#pragma unroll
    for (int t = 0; t < K; ++t) {
        dist[t] = t < pad ? -kInf : kInf;
        idx[t] = -1;
    }
    float bound2 = a.bound == KNN_BOUND_NONE ? kInf : seed2;  // B(leaf)^2 (both leaves' lanes)
    float lim = bound2;  // min(D_p[k]^2, B^2): what a candidate must beat
    uint32_t n_score = 0, n_tiles = 0, n_ins = 0, n_pass = 0, n_cand = 0;
    uint64_t n_pairs = 0;

    // this lane's value and its partner's, as (leaf 0's query jj, leaf 1's
    // query jj): what column jj of the two products is compared with
    auto both = [&](float v, float &v0, float &v1) {
        const float o = __shfl_xor(v, 32);
        v0 = hh ? o : v;
        v1 = hh ? v : o;
    };
    // bounds after a change of the lists: B1, B2 over the leaf, B(Par) over
    // the pair; the parts exchange their k-th distances first
    auto refresh = [&]() __attribute__((always_inline)) {
        float kth = dist[K - 3];
        if (parts) {
            const uint32_t mine = __float_as_uint(fmaxf(kth, 0.f));
            const uint32_t old = atomicMin(&s_kth[lane], mine);
            kth = __uint_as_float(min(mine, old));
        }
        if (a.bound != KNN_BOUND_NONE) {
            float b = reduce32(valid ? kth : -kInf, OpMax());  // B1^2
            if (a.bound == KNN_BOUND_B) {
                float lo = reduce32(valid ? kth : kInf, OpMin());
                const float b2 = __builtin_amdgcn_sqrtf(lo) + lam2;
                b = fminf(b, b2 * b2);
                lo = xor32_op(lo, OpMin());
                const float bp = __builtin_amdgcn_sqrtf(lo) + lam2_anc;
                b = fminf(b, bp * bp);
            }
            bound2 = fminf(fminf(b, seed2), bound2);
        }
        lim = fminf(kth, bound2);
    };
    const __bf16 *abf = reinterpret_cast<const __bf16 *>(a.sw_abf);
    const __bf16 *cbf = reinterpret_cast<const __bf16 *>(a.sw_cbf);

    // the rows of a leaf in `mask` (this half's 16 bits, then the other's),
    // one per lane and round: the distance in FP64, then the list
    auto insert_rows = [&](int leaf, int base, uint32_t mask) __attribute__((always_inline)) {
        n_cand += __popc(mask);
        const float *rows = a.rlpts + int64_t(leaf) * a.r_leaf_slots * DP;
#pragma unroll 1
        for (int pass = 0; pass < 32; ++pass) {
            const bool has = mask != 0;
            if (!ballot(has)) break;
            ++n_pass;
            const int b = has ? __builtin_ctz(mask) : 0;
            mask &= mask - 1u;
            const int rb16 = b & 15, hb = b < 16 ? hh : 1 - hh;
            const int row = 8 * (rb16 >> 2) + 4 * hb + (rb16 & 3);
            const float x0 = (float)d2_fp64_rows<DP>(my_q, rows + (has ? row : 0) * DP);
            const float x = has ? x0 : kInf;
            n_ins += (x < dist[K - 1]) ? 1u : 0u;
            sorted_insert<K>(dist, idx, x, base + row);
        }
        refresh();
    };
    // whether the tiles' margin covers every query and row of a block
    auto covered = [&](float qlen, float rcb) __attribute__((always_inline)) -> bool {
        return rcb < 0.5f * kTileLong &&
               !ballot(valid && !(qlen >= kTileShort && qlen < 0.5f * kTileLong));
    };
    // the block of a step (-1: none there, -2: no block from here on is needed)
    auto block_of = [&](int st) __attribute__((always_inline)) -> int {
        int rb;
        if (use_sort) {
            rb = uniform_i(int(s_order[st]));
        } else {
            const int off = (st + 1) >> 1;
            rb = (st & 1) ? sblock + off : sblock - off;
            if (rb < 0 || rb >= n_blocks) return -1;
        }
        if (parts) refresh();
        if (use_sort && a.bound != KNN_BOUND_NONE) {
            // no query of this wave needs a block whose key exceeds its bound
            // plus R; the keys ascend (R and the keys are sums of squares: below
            // 2^-40 they may have lost their bits)
            const float bw = uniform_f(reduce64(valid ? lim : -kInf, OpMax()));
            const float bmax =
                bw < kInf ? __builtin_amdgcn_sqrtf(fmaxf(bw, 0.f)) * (1.0f + 0x1p-20f) : kInf;
            if (uniform_f(s_okey[st]) > fmaxf((bmax + R) * kSlack, 0x1p-40f)) return -2;
        }
        return rb;
    };
    // query operands of a block: q - C_B of column jj of both leaves at this
    // lane's dimensions; returns |q - C_B|^2 of this lane's query
    auto operands = [&](int rb, bf16x8_t (&bq0)[S], bf16x8_t (&bq1)[S])
                        __attribute__((always_inline)) -> float {
        const float *cb = a.sw_bcen + int64_t(rb) * DP;
        float n0 = 0.f, n1 = 0.f;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const float4 c0 = *reinterpret_cast<const float4 *>(cb + s * 16 + hh * 8);
            const float4 c1 = *reinterpret_cast<const float4 *>(cb + s * 16 + hh * 8 + 4);
            const float cv[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const float *xr = rows_w + (32 * g + jj) * L::row + s * 16 + hh * 8;
                const float4 x0 = *reinterpret_cast<const float4 *>(xr);
                const float4 x1 = *reinterpret_cast<const float4 *>(xr + 4);
                const float xv[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float df = xv[e] - cv[e];
                    if (g == 0) {
                        n0 = fmaf(df, df, n0);
                        bq0[s][e] = (__bf16)df;
                    } else {
                        n1 = fmaf(df, df, n1);
                        bq1[s][e] = (__bf16)df;
                    }
                }
            }
        }
        return (hh ? n1 : n0) + __shfl_xor(hh ? n0 : n1, 32);
    };
    bool left = false;  // blocks left for the pass below

    for (int st = parts ? w : 0; st < n_steps && n_valid > 0; st += parts ? 4 : 1) {
        const int rb = block_of(st);
        if (rb == -2) break;
        if (rb < 0) continue;
        bf16x8_t bq0[S], bq1[S];
        const float qnb = operands(rb, bq0, bq1);
        const float qlenb = sqrtf(qnb);
        const int L0 = rb * NB;
        const float rcb = uniform_f(a.sw_rcb[rb]);
        if (!covered(qlenb, rcb)) {
            left = true;
            continue;
        }
        uint32_t own;  // the block's leaves that some query of the wave keeps
        {
            f32x16_t acc0, acc1;
            float lam[16];
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const float4 v = *reinterpret_cast<const float4 *>(a.sw_cn + L0 + g4 * 8 + hh * 4);
                const float4 l = *reinterpret_cast<const float4 *>(a.sw_lam + L0 + g4 * 8 + hh * 4);
                acc0[g4 * 4 + 0] = v.x;
                acc0[g4 * 4 + 1] = v.y;
                acc0[g4 * 4 + 2] = v.z;
                acc0[g4 * 4 + 3] = v.w;
                lam[g4 * 4 + 0] = l.x;
                lam[g4 * 4 + 1] = l.y;
                lam[g4 * 4 + 2] = l.z;
                lam[g4 * 4 + 3] = l.w;
            }
            acc1 = acc0;
            const __bf16 *arow = cbf + int64_t(L0) * DP + (hh * 32 + jj) * 8;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const bf16x8_t ar = *reinterpret_cast<const bf16x8_t *>(arow + s * 512);
                acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ar, bq0[s], acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ar, bq1[s], acc1, 0, 0, 0);
            }
            // idle lanes: a zero bound against a low end of +inf keeps nothing
            const float low = valid ? qnb - bf16_margin<DP>(qlenb, rcb) : kInf;
            const float bp = !valid      ? 0.f
                             : lim < kInf ? __builtin_amdgcn_sqrtf(fmaxf(lim, 0.f)) * (1.0f + 0x1p-20f)
                                          : kInf;
            float low0, low1, bp0, bp1;
            both(low, low0, low1);
            both(bp, bp0, bp1);
            // bit r: the sign of (b_p + rho)^2 (1 + 2^-16) - low end clear in
            // either product (keep); then nibble g moves to rows 8 g + 4 h ..
            uint32_t m16 = 0;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float t0 = bp0 + lam[r], t1 = bp1 + lam[r];
                const uint32_t k0 = __float_as_uint(fmaf(t0 * kSlack, t0, -(acc0[r] + low0)));
                const uint32_t k1 = __float_as_uint(fmaf(t1 * kSlack, t1, -(acc1[r] + low1)));
                m16 |= (~(k0 & k1) >> 31) << r;
            }
            uint32_t m =
                (m16 & 0xfu) | ((m16 & 0xf0u) << 4) | ((m16 & 0xf00u) << 8) | ((m16 & 0xf000u) << 12);
            m <<= 4 * hh;
            if (a.bound == KNN_BOUND_NONE) m = 0xffffffffu;
            const float mf = reduce64(__builtin_bit_cast(float, m), OpOrBits());
            const uint32_t vrows = uint32_t(ballot(lane < 32 && a.sw_cn[L0 + jj] < kInf));
            own = uint32_t(uniform_i(__builtin_bit_cast(int, mf))) & vrows;
            n_score += __popc(vrows);
        }
        if (!own) continue;
        // what column jj's values are compared with: D < base + margin, base
        // = min(D_p[k], B)^2 (1 + 2^-16) - |q - C_B|^2 (-inf for idle lanes)
        float qlen0, qlen1, base0, base1;
        both(qlenb, qlen0, qlen1);
        both(valid ? lim * kSlack - qnb : -kInf, base0, base1);
        struct TileIn {
            bf16x8_t ar[S];
            float rnj;  // |r_j - C_B|^2 of row j = lane % 32
            int2 rr;
            float rl;
        };
        auto tload = [&](int leaf, TileIn &t) {
            const __bf16 *arow = abf + int64_t(leaf) * NB * DP + (hh * 32 + jj) * 8;
#pragma unroll
            for (int s = 0; s < S; ++s) t.ar[s] = *reinterpret_cast<const bf16x8_t *>(arow + s * 512);
            t.rnj = a.sw_rn[int64_t(leaf) * NB + jj];
            t.rr = a.rrange[a.r_first_leaf + leaf];
            t.rl = a.sw_rlen[leaf];
        };
        auto tile = [&](int leaf, const TileIn &t) __attribute__((always_inline)) {
            const int base = uniform_i(t.rr.x);
            const int cnt = uniform_i(t.rr.y);
            ++n_tiles;
            n_pairs += uint64_t(cnt) * uint64_t(n_valid);
            const f32x16_t accn = bf16_norm_init(t.rnj, t.rnj < kInf, hh);
            f32x16_t acc0 = accn, acc1 = accn;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(t.ar[s], bq0[s], acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(t.ar[s], bq1[s], acc1, 0, 0, 0);
            }
            // (strict: the margin is 1.25 times the proven bound; capped at
            // FLT_MAX: rows past the leaf hold +inf and never pass)
            const float rl = uniform_f(t.rl);
            const float thr0 = fminf(base0 + bf16_margin<DP>(qlen0, rl), 0x1.fffffep127f);
            const float thr1 = fminf(base1 + bf16_margin<DP>(qlen1, rl), 0x1.fffffep127f);
            float am0 = acc0[0], am1 = acc1[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) {
                am0 = fminf(am0, acc0[r]);
                am1 = fminf(am1, acc1[r]);
            }
            if (!ballot(am0 < thr0 || am1 < thr1)) return;
            // bit r: the sign of D - thr; each lane keeps the rows of its half
            // for its own query and takes the other half's from lane ^ 32
            uint32_t mk0 = 0, mk1 = 0;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                mk0 |= (__float_as_uint(acc0[r] - thr0) >> 31) << r;
                mk1 |= (__float_as_uint(acc1[r] - thr1) >> 31) << r;
            }
            insert_rows(leaf, base,
                        (hh ? mk1 : mk0) | (uint32_t(__shfl_xor(int(hh ? mk0 : mk1), 32)) << 16));
            both(valid ? lim * kSlack - qnb : -kInf, base0, base1);
        };
        // software-pipelined over the kept leaves: the next one's operands
        // are loaded while the current one is multiplied (two register sets
        // in turn; past the last leaf the loads repeat the current one)
        auto next = [&](int prev, bool &more) -> int {
            more = own != 0;
            const int c = more ? __builtin_ctz(own) : prev;
            own &= own - 1u;
            return c;
        };
        TileIn t0, t1;
        bool m1, m2;
        int c0 = __builtin_ctz(own);
        own &= own - 1u;
        tload(L0 + c0, t0);
        for (;;) {
            const int c1 = next(c0, m1);
            tload(L0 + c1, t1);
            tile(L0 + c0, t0);
            if (!m1) break;
            const int c2 = next(c1, m2);
            tload(L0 + c2, t0);
            tile(L0 + c1, t1);
            if (!m2) break;
            c0 = c2;
        }
    }

    // the blocks that the margin does not cover: leaves scored by their boxes,
    // rows filtered by FP32 differences
    for (int st = parts ? w : 0; __builtin_expect(left, 0) && st < n_steps; st += parts ? 4 : 1) {
        const int rb = block_of(st);
        if (rb == -2) break;
        if (rb < 0) continue;
        bf16x8_t unused0[S], unused1[S];  // (the same sum as above: the same decision)
        if (covered(sqrtf(operands(rb, unused0, unused1)), uniform_f(a.sw_rcb[rb]))) continue;
        const int L0 = rb * NB;
        uint32_t rest = uint32_t(ballot(lane < 32 && a.sw_cn[L0 + jj] < kInf));
        n_score += __popc(rest);
        for (; rest; rest &= rest - 1u) {
            const int leaf = L0 + __builtin_ctz(rest);
            const float *b = a.rbox + int64_t(a.r_first_leaf + leaf) * 2 * DP;
            float sd = 0.f;
#pragma unroll 4
            for (int u = 0; u < DP; ++u) {
                const float gap = fmaxf(fmaxf(b[u] - my_q[u], my_q[u] - b[DP + u]), 0.0f);
                sd = fmaf(gap, gap, sd);
            }
            if (!ballot(valid && (a.bound == KNN_BOUND_NONE || !(sd > lim * kSlack)))) continue;
            const int2 rr = a.rrange[a.r_first_leaf + leaf];
            const int base = uniform_i(rr.x), cnt = uniform_i(rr.y);
            ++n_tiles;
            n_pairs += uint64_t(cnt) * uint64_t(n_valid);
            const float *rows = a.rlpts + int64_t(leaf) * a.r_leaf_slots * DP;
            const float thr = valid ? lim * kSlack * (1.0f + (DP + 6) * 0x1p-24f) : -1.0f;
            uint32_t near = 0;
#pragma unroll 1
            for (int r = 0; r < cnt; ++r) {
                float x = 0.f;
#pragma unroll 4
                for (int u = 0; u < DP; ++u) {
                    const float df = my_q[u] - rows[r * DP + u];
                    x = fmaf(df, df, x);
                }
                near |= uint32_t(x <= thr && x < kInf) << r;
            }
            if (ballot(near != 0))
                insert_rows(leaf, base, half_bits(near, hh) | (half_bits(near, 1 - hh) << 16));
        }
    }

    // parts: the first wave takes over the others' lists, one after another
    // (ascending, so it stops at the first entry that beats no lane's last)
    if (parts) {
        float *s_d = reinterpret_cast<float *>(smem + L::off_list);
        int *s_i = reinterpret_cast<int *>(s_d + 64 * K);
        for (int ww = 1; ww < 4; ++ww) {
            __syncthreads();
            if (w == ww) {
#pragma unroll
                for (int t = 0; t < K; ++t) {
                    s_d[t * 64 + lane] = dist[t];
                    s_i[t * 64 + lane] = idx[t];
                }
            }
            __syncthreads();
            if (w == 0) {
#pragma unroll 1
                for (int t = pad; t < K; ++t) {
                    const float x = s_d[t * 64 + lane];
                    if (!ballot(x < dist[K - 1])) break;
                    sorted_insert<K>(dist, idx, x, s_i[t * 64 + lane]);
                }
            }
        }
    }

    // ---- write-out -----------------------------------------------------------
    float worst = -1.0f;
    const bool writer = !parts || w == 0;
    if (writer && n_valid > 0) {
        // the query's own point leaves the list
        if (a.self) {
            bool found = false;
#pragma unroll
            for (int t = 0; t < K; ++t) {
                found = found || (idx[t] == qpos && idx[t] >= 0);
                if (found) {
                    dist[t] = t + 1 < K ? dist[t + 1] : kInf;
                    idx[t] = t + 1 < K ? idx[t + 1] : -1;
                }
            }
        }
        const int last = pad + a.k - 1;  // slot of the k-th entry
        if (a.walk_ties) {
            // equal distances at the k-th place: in the order of the walk,
            // whose slots hold one leaf at stride 64
            const int ng_log2 = DP == 64 ? 0 : 6 - a.lpl_log2;
            float xk = 0.f, xn = 0.f;
#pragma unroll
            for (int t = 0; t + 1 < K; ++t) {
                xk = t == last ? dist[t] : xk;
                xn = t == last ? dist[t + 1] : xn;
            }
            uint64_t tied = ballot(valid && xk == xn && xk < kInf);
            while (tied) {
                const int src = __builtin_ctzll(tied);
                tied &= tied - 1;
                const float xs = __shfl(xk, src);
                const int ql = uniform_i(__shfl(qleaf, src));
                // bubble passes over the tied entries of that lane's list
                for (int it = 0; it < K; ++it) {
                    bool swapped = false;
#pragma unroll
                    for (int t = 0; t + 1 < K; ++t) {
                        const float d0 = __shfl(dist[t], src), d1 = __shfl(dist[t + 1], src);
                        if (d0 == xs && d1 == xs) {
                            const int i0 = uniform_i(__shfl(idx[t], src)),
                                      i1 = uniform_i(__shfl(idx[t + 1], src));
                            if (walk_meets_second_first<DP>(a, i0, i1, ql, ng_log2)) {
                                swapped = true;
                                if (lane == src) {
                                    idx[t] = i1;
                                    idx[t + 1] = i0;
                                }
                            }
                        }
                    }
                    if (!swapped) break;
                }
            }
        }
        // output keys: the FP32 distance from FP64 and the original index;
        // slots that hold no entry (and, after the choice above, the ones past
        // the k-th) rank last
#pragma unroll
        for (int t = 0; t < K; ++t) {
            const bool real = valid && idx[t] >= 0 && (!a.walk_ties || t <= last);
            const int p = real ? idx[t] : 0;
            float key = t < pad ? -kInf : kInf;
            int o = 0x7fffffff - K + t;
            if (real) {
                key = (float)sqrt(d2_fp64_rows<DP>(my_q, a.rpts + int64_t(p) * DP));
                o = a.rperm[p];
            }
            dist[t] = key;
            idx[t] = o;
        }
        // the list is ascending but for equal keys: exchange neighbours until
        // (key, index) is in order everywhere
        for (int it = 0; it < K; ++it) {
            bool swapped = false;
#pragma unroll
            for (int par = 0; par < 2; ++par)
#pragma unroll
                for (int t = par; t + 1 < K; t += 2) {
                    const bool sw =
                        dist[t + 1] < dist[t] || (dist[t + 1] == dist[t] && idx[t + 1] < idx[t]);
                    const float d0 = dist[t], d1 = dist[t + 1];
                    const int i0 = idx[t], i1 = idx[t + 1];
                    dist[t] = sw ? d1 : d0;
                    dist[t + 1] = sw ? d0 : d1;
                    idx[t] = sw ? i1 : i0;
                    idx[t + 1] = sw ? i0 : i1;
                    swapped |= sw;
                }
            if (!ballot(swapped)) break;
        }
        if (valid) {
            const int64_t row = int64_t(a.qperm[qpos]) * a.k - pad;
#pragma unroll
            for (int t = 0; t < K; ++t) {
                if (t >= pad && t <= last) {
                    a.out_idx[row + t] = idx[t] >= 0x7fffffff - K ? -1 : idx[t];
                    a.out_dist[row + t] = dist[t];
                    if (t == last) worst = dist[t];
                }
            }
        }
    }
    bool fb = false;
    if (writer && a.seed && valid) fb = !((double)worst * worst <= (double)seed2 * (1.0 - 0x1p-20));
    const float lw = reduce32(worst, OpMax());
    const float fl = reduce32(fb ? 1.0f : 0.0f, OpMax());
    const float fbb = reduce32((valid && worst < kInf) ? worst : kInf, OpMin());
    const uint64_t fbmask = ballot(fb);
    if (writer && jj == 0 && has_leaf) {
        if (a.leaf_kth) a.leaf_kth[qleaf] = fmaxf(lw, 0.0f);
        if (a.fallback && fl > 0.f) {
            a.fallback[qleaf] = 1;
            if (a.fb_bound) a.fb_bound[qleaf] = fbb < kInf ? (fbb + lam2) * (1.0f + 0x1p-20f) : kInf;
        }
    }
    if (a.wave_log || a.stats) {
        int ins = n_ins, cand = int(n_cand);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            ins += __shfl_xor(ins, off);
            cand += __shfl_xor(cand, off);
        }
        if (a.wave_log && lane == 0) {
            uint32_t *wl = a.wave_log + (int64_t(blockIdx.x) * 4 + w) * 8;
            wl[0] = 0;
            wl[1] = n_score;
            wl[2] = n_tiles;
            wl[3] = uint32_t(ins);
            wl[4] = n_pass;
            wl[5] = uint32_t(leaf0 + 2 * w);
            wl[7] = uint32_t(cand);
        }
        if (a.stats && lane == 0) {
            atomicAdd(&a.stats[ST_SCORE], (unsigned long long)n_score);
            atomicAdd(&a.stats[ST_TILES], (unsigned long long)n_tiles);
            atomicAdd(&a.stats[ST_PAIRS], (unsigned long long)n_pairs);
            atomicAdd(&a.stats[ST_INSERTS], (unsigned long long)ins);
            atomicAdd(&a.stats[ST_FB_QUERIES], (unsigned long long)__popcll(fbmask));
        }
    }
}

// list lengths: the smallest that holds kk + 2 entries (kk <= 64).  They hold k =
// 8, 16, 32, 50 and 64 (or that many with the query's own point: 53 = 51 + 2); a
// list costs two registers an entry, and 53 is the longest of them that leaves
// room for two waves per SIMD (256 registers, some 75 in scratch); 66 has one
// wave per SIMD and nothing in scratch.
template <int DP>
hipError_t launch_search_pair(const SearchArgs &a, int kk, int grid, hipStream_t s) {
    if (!a.sw_abf || a.r_leaf_slots > 32) return hipErrorInvalidValue;
    const int need = kk + 2;
    if (need <= 10)
        k_search_pair<DP, 10><<<grid, 256, 0, s>>>(a);
    else if (need <= 18)
        k_search_pair<DP, 18><<<grid, 256, 0, s>>>(a);
    else if (need <= 34)
        k_search_pair<DP, 34><<<grid, 256, 0, s>>>(a);
    else if (need <= 53)
        k_search_pair<DP, 53><<<grid, 256, 0, s>>>(a);
    else if (need <= 66)
        k_search_pair<DP, 66><<<grid, 256, 0, s>>>(a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace knnx
