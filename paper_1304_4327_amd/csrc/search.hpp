// Search-side declarations shared by the traversal kernels and the host code.
#pragma once

#include "common.hpp"

#include <algorithm>

namespace knnx {

// counters accumulated by the traversal kernels (uint64 each)
enum StatSlot {
    ST_SCORE = 0,
    ST_TILES = 1,
    ST_PAIRS = 2,
    ST_INSERTS = 3,
    ST_FB_QUERIES = 4,
    ST_COUNT = 8
};

struct SearchArgs {
    // reference tree
    const float *rpts;
    const int32_t *rperm;
    const int2 *rrange;
    const float *rbox;
    const float *rlam;
    const float *rlpts;  // leaf-blocked points (r_leaf_slots per leaf)
    int r_leaf_slots;
    int r_first_leaf;
    // query tree
    const float *qpts;
    const int32_t *qperm;
    const int2 *qrange;
    const float *qbox;
    const float *qlam;
    int q_first_leaf;
    int q_n_leaves;
    // leaves to process: active == NULL means all; otherwise only leaves
    // with active[leaf] != 0 (the waves keep their sibling-aligned leaves)
    const int *active;
    // launch order of the wave slots (largest leaf radius first), or NULL:
    // wave i of the launch takes slot order[i]
    const int *order;
    int split;  // log2 of the waves that share one slot's queries (split_for)
    int d, k, lpl_log2;
    int bound;          // knn_bound
    int self;           // exclude reference position == query position
    int walk_ties;      // FP32 requests: among equal distances the plain walk's order
    const float *seed;  // per query leaf, or NULL
    int64_t *out_idx;
    float *out_dist;
    float *leaf_kth;    // per query leaf, or NULL
    int *fallback;      // per query leaf flag (seeded runs), or NULL
    float *fb_bound;    // per query leaf (seeded runs): a proven bound for the
                        // fallback pass, min D_p[k] + 2 lambda over the leaf's
                        // queries with a full list (+inf if none), or NULL
    unsigned long long *stats;  // ST_COUNT counters, or NULL; the FP32 kernel with a
                                // seed adds its second pass's counts to the next
                                // ST_COUNT
    // sweep with two query leaves per wave (k_search_pair): the
    // reference side of every tile and block Score, centred on the centre
    // C_B of the leaf's block (subtree of 32 leaves), made once per search
    // by k_wsweep_prep.  Leaves are padded to whole blocks.  An operand's 8
    // dimensions 16 s + 8 h .. of 32 rows are 512 contiguous bytes.
    const uint16_t *sw_abf;  // [leaf][s][h][32 rows][8] bf16(-2 (r - C_B)), 0 past the leaf
    const float *sw_rn;      // [leaf][32] |r - C_B|^2 (FP32, finite), +inf past the leaf
    const float *sw_rlen;    // [leaf] largest |r - C_B|, rounded up
    const uint16_t *sw_cbf;  // [block][s][h][32 leaves][8] bf16(-2 (C_L - C_B)), C_L the leaf's ball centre
    const float *sw_cn;      // [leaf] |C_L - C_B|^2 (finite), +inf for empty or padding leaves
    const float *sw_lam;     // [leaf] radius of the leaf's ball, 0 for padding
    const float *sw_bcen;    // [block][DP] C_B
    const float *sw_rcb;     // [block] largest |C_L - C_B| of the block, rounded up; +inf
                             // where a norm of the block is beyond the tiles' range
    uint32_t *wave_log;         // debug: 8 words per wave (ticks, scores, tiles, inserts, passes, leaf,
                                // staged tiles of the d = 64 sweep, candidates of the BF16 filters)
    // Score log of the debug kernel (launch_search_valu_debug_d3): one
    // record of kDbgWords words per Score call, or NULL; and the visit order
    // (0: nearer child first, 1: farther child first)
    uint32_t *dbg_log;
    unsigned int *dbg_count;  // records written (may exceed dbg_cap: then truncated)
    int dbg_cap;              // capacity in records
    int far_first;
    // tile list of the debug kernel: with tile_replay == 0 each wave records
    // the reference leaves it evaluates (tile_log[wave * tile_cap + i], the
    // count in tile_cnt[wave]); with tile_replay == 1 it evaluates exactly
    // those leaves in that order, without the walk
    uint32_t *tile_log;
    uint32_t *tile_cnt;
    int tile_cap;
    int tile_replay;
};

// Score-log record: node, kept (1/0), first query leaf of the wave, number
// of leaves of the wave, then the squared bound B(N_q)^2 of each leaf (as
// FP32 bits) at the time of the call
constexpr int kDbgWords = 12;
constexpr int kDbgMaxLeaves = kDbgWords - 4;

// per-dimension launchers (search_d*.hip): D computed dimensions (d for
// d <= 4, else d rounded up to 8, 16, 32 or 64 with zero padding); K is
// the compile-time list length
hipError_t launch_search_valu_d1(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_valu_d2(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_valu_d3(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_valu_d4(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_valu_d8(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_valu_d16(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_valu_d32(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_valu_d64(const SearchArgs &a, int K, int grid, hipStream_t s);
// the same with a seed radius (search_seeded_d*.hip)
hipError_t launch_search_valu_seeded_d1(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_valu_seeded_d2(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_valu_seeded_d3(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_valu_seeded_d4(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_valu_seeded_d8(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_valu_seeded_d16(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_valu_seeded_d32(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_valu_seeded_d64(const SearchArgs &a, int K, int grid, hipStream_t s);

// the d = 3 FP32 kernel with the Score log and the visit-order switch
// (search_debug_d3.hip); lists up to 16
hipError_t launch_search_valu_debug_d3(const SearchArgs &a, int K, int grid, hipStream_t s);

// the traversal kernel with BF16 matrix-core BaseCase tiles
// (search_mt_d*.hip): 16 or 32 computed dimensions, two query leaves per wave
// (lpl_log2 = 5), reference leaves of <= 32 points, K <= 16; the seeded form
// when a.seed is set
// (stride 8 in the plain form only)
// references from which FP32 requests use them
constexpr int64_t kTilePoints = 2048;
hipError_t launch_search_mt_d8(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_mt_d16(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_mt_d32(const SearchArgs &a, int K, int grid, hipStream_t s);

// one query per wave (search_few.hip): strides up to 16, every pruning bound
// but KNN_BOUND_NONE, no seed, no counters; lists of kk <= kFewList entries.
// The slot-per-wave walk lasts as long as its slowest wave until the chip is
// full, and a slot's queries open the more of the reference tree the sparser
// they lie in it; one query per wave costs the same per query throughout, about
// 1.6 us a thousand at d = 3, 2 to 4 at d = 5, 6 to 15 at d = 8.
// Measured (us, one query per wave / slot walk; k = 10, 32 points a leaf):
//   mixtures, d = 3: 128,000 queries of 10,000 points 207 / 182, 256,000 of
//   200,000 453 / 447, 512,000 of 1M 814 / 1031; d = 8: 128,000 of 10,000
//   773 / 655, 256,000 of 200,000 3885 / 6400; d = 13: 66,000 of 10,000 and of
//   40,000 343 / 1332 and 714 / 3315; a manifold, d = 13: 128,000 of 10,000
//   605 / 412, of 200,000 1002 / 1314
//   uniform, d = 2: 64,000 of 10,000 107 / 82, of 200,000 104 / 202; d = 3:
//   64,000 of 10,000 116 / 137, 256,000 of 200,000 439 / 313; d = 13: 32,000 of
//   10,000 1591 / 1450, 64,000 of 10,000 2960 / 1495, of 200,000 13.5 / 14.7 ms
//   d = 1: 40,000 of 3000 66 / 52, of 150,000 73 / 114
//   any d: 40,000 of 100 50 to 100 / 40 to 85, of 1000 52 to 90 / 50 to 210
// So the line lies lower where every kind of data crosses early (d = 1, d = 2,
// few references) and up to d = 8 inside what uniform sets bear; above d = 8,
// where uniform sets cross at 30,000 to 70,000 queries and clustered ones gain
// three times as much as those lose, between the two.  Lists of more than 16
// entries cost the slot walk several times as much (40,000 queries of 1000, d =
// 3, k = 40: 111 / 609), whatever the rest.
constexpr int kFewList = 62;
inline bool few_queries(int64_t n_q, int64_t n_ref, int d, int kk) {
    const int64_t most = 65536 + n_ref / (d <= 4 ? 6 : d <= 8 ? 2 : 8);
    if (kk > 16) return n_q <= most;
    const int64_t line = d == 1   ? 24576 + n_ref / 8
                         : d == 2 ? std::min(most, 32768 + n_ref / 2)
                                  : most;
    return n_q <= std::min(line, 16384 + 48 * n_ref);
}
hipError_t launch_search_few_d(const SearchArgs &a, int d, int64_t n_q, hipStream_t s);

// the sweep with two query leaves per wave (search_pair_d32.hip, _d64.hip): the
// operands of launch_wsweep_prep, lists of kk <= 64 entries
// references from which FP32 requests use it
constexpr int64_t kSweepPoints = 3000;
constexpr int kPairLeaves = 8;  // query leaves per workgroup (two per wave)
// parts: one pair of leaves per workgroup, its four waves dealing the blocks
inline int pair_grid(int n_leaves, bool parts) {
    const int per = parts ? 2 : kPairLeaves;
    return (n_leaves + per - 1) / per;
}
// (256 CUs, two workgroups on each)
inline bool pair_parts(int n_leaves) { return pair_grid(n_leaves, false) <= 256; }
hipError_t launch_search_pair_dp32(const SearchArgs &a, int kk, hipStream_t s);
hipError_t launch_search_pair_dp64(const SearchArgs &a, int kk, hipStream_t s);

// reference leaves the d = 64 sweep scores together (one subtree)
constexpr int kSweepBlock = 32;

// reference-side operands of the two-leaf sweep, strides 32 and 64 (see the
// sw_* fields): fills them for the n_blocks * 32 (padded) leaves of the
// reference tree in args
hipError_t launch_wsweep_prep(const SearchArgs &args, int dp, uint16_t *abf, float *rn, float *rlen,
                              uint16_t *cbf, float *cn, float *lam, float *bcen, float *rcb,
                              hipStream_t s);

// BF16 MFMA kernels (search_mfma_d*.hip), stride 16, 32 or 64
hipError_t launch_search_mfma_dp16(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_mfma_dp32(const SearchArgs &a, int K, int grid, hipStream_t s);
hipError_t launch_search_mfma_dp64(const SearchArgs &a, int K, int grid, hipStream_t s);

// Waves per slot of query leaves, as a power of two.  A small query set has
// fewer slots than the chip has SIMDs, and then the call lasts as long as one
// wave's walk, which grows with the queries it carries (each of them opens
// its own part of the reference tree).  The queries of a slot are then dealt
// over 1 << split waves, as long as every wave has a SIMD to itself: beyond
// that (4096 waves were tried) the repeated walks cost up to three times what
// the shorter ones save.  Every query sees the reference nodes in the same
// order as in the undivided slot: the visit-order key still comes from the
// whole slot.
constexpr int kSplitWaves = 1024;
inline int split_for(int64_t slots, int lg, int max_leaf) {
    int most = 6 - lg;  // one leaf per wave, then down to one query
    while ((1 << (most - (6 - lg))) < max_leaf) ++most;
    int s = 0;
    while (s < most && (slots << (s + 1)) <= kSplitWaves) ++s;
    return s;
}

// zero n 32-bit words with a kernel (api.hip)
hipError_t zero_words(void *p, int64_t n, hipStream_t s);

// exclusive prefix sums (scan.hip): out[0] = 0, out[i + 1] = in[0] + ... +
// in[i] for 1 <= n <= kScanMax; tops is scratch of scan_scratch(n) values
constexpr int64_t kScanMax = int64_t(1) << 24;
int64_t scan_scratch(int64_t n);
hipError_t exclusive_scan(const int64_t *in, int64_t n, int64_t *out, int64_t *tops,
                          hipStream_t s);

// k-furthest-neighbour kernels (search_far_d*.hip), stride 4 .. 64, lists of
// kk <= 64 entries
hipError_t launch_search_far_dp4(const SearchArgs &a, int kk, int grid, hipStream_t s);
hipError_t launch_search_far_dp8(const SearchArgs &a, int kk, int grid, hipStream_t s);
hipError_t launch_search_far_dp16(const SearchArgs &a, int kk, int grid, hipStream_t s);
hipError_t launch_search_far_dp32(const SearchArgs &a, int kk, int grid, hipStream_t s);
hipError_t launch_search_far_dp64(const SearchArgs &a, int kk, int grid, hipStream_t s);

// compile-time list lengths; a request for a list of kk entries (k, or k+1
// when the query's own point shares the list) uses the smallest K >= kk
constexpr int kListSizes[] = {4, 5, 8, 10, 11, 16, 32, 50, 51, 64};
inline int list_size_for(int kk) {
    for (int K : kListSizes)
        if (K >= kk) return K;
    return -1;
}

}  // namespace knnx
