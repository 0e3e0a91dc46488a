// kd-tree construction on the GPU (Section "Space Trees": Definition 1 and the
// kd-tree bounds paragraph; points live only in leaves, as in the discussion of
// Gray's AllNN).
//
// Split rule (the paper fixes none; this is the library's):
//   complete tree of depth L = smallest L with ceil(n / 2^L) <= leaf_size,
//   heap-ordered nodes; node ranges are data independent (left child gets
//   floor(c/2) of its parent's c points).  A node splits on the dimension of
//   largest FP32 box extent (ties -> lowest); its left child receives the
//   floor(c/2) smallest points under (coordinate, original index); both
//   children keep ascending original-index order (stable partition).
//
// Level-synchronous construction, two regimes:
//   * levels whose segments exceed what one workgroup can hold run as
//     grid-wide passes over a copy of the points kept in the current order,
//     one array per dimension (a pass over the split dimension reads 4 bytes a
//     point, whatever d; each partition moves all dimensions and gathers the
//     children's boxes on the way): radix select (up to 11-bit digits of an
//     order-preserving uint32 key) of the median key per segment, and a
//     stable partition by a segmented scan of (less, equal) counts;
//   * one workgroup builds the whole subtree of a segment it can hold
//     (k_seg_build): the points in LDS up to 16 dimensions, else read in place.
//     Several waves share a node while there are fewer nodes than waves, then
//     each node is one wave's work.  The same launch writes the points in tree
//     order (FP32, padded to dp) and leaf-blocked, the leaf boxes, the exact
//     leaf lambda (FP64, rounded up) and the subtree's internal lambda.
// A set of up to a few thousand points is one launch, or two: the first splits
// it into segments of about a thousand points, so that more than one
// workgroup finishes it.
#include "common.hpp"

#include <condition_variable>
#include <functional>
#include <mutex>
#include <thread>

#include <algorithm>
#include <atomic>
#include <type_traits>
#include <vector>

namespace knnx {
namespace {

// elements per block in grid-wide levels: histograms, and the partition with
// its counts (shorter: more waves in flight to cover its loads)
constexpr int kHistChunk = 2048, kMoveChunk = 1024;
constexpr int kBlock = 256;

struct Sel {
    uint32_t prefix, mask;  // key bits fixed so far
    int32_t rank;           // rank still wanted among keys matching the prefix
    int32_t bits;           // low bits not yet fixed (0: the median key is known)
};

__device__ inline uint64_t lanemask_lt() {
    return (uint64_t(1) << (threadIdx.x & 63)) - 1;
}
__device__ inline int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

// minimum / maximum of unsigned keys over the wave by lane moves alone
// (complete in lane 63): within rows of 16, then each row's last lane to the
// next row, then to the upper half
template <int CTRL, int ROWS>
__device__ inline uint32_t dpp_u(uint32_t identity, uint32_t v) {
    return uint32_t(__builtin_amdgcn_update_dpp(int(identity), int(v), CTRL, ROWS, 0xF, false));
}
__device__ inline uint32_t wave_umin(uint32_t v) {
    v = min(v, dpp_u<0x111, 0xF>(~0u, v));  // row_shr:1, 2, 4, 8
    v = min(v, dpp_u<0x112, 0xF>(~0u, v));
    v = min(v, dpp_u<0x114, 0xF>(~0u, v));
    v = min(v, dpp_u<0x118, 0xF>(~0u, v));
    v = min(v, dpp_u<0x142, 0xA>(~0u, v));  // row_bcast:15
    v = min(v, dpp_u<0x143, 0xC>(~0u, v));  // row_bcast:31
    return v;
}
__device__ inline uint32_t wave_umax(uint32_t v) {
    v = max(v, dpp_u<0x111, 0xF>(0u, v));
    v = max(v, dpp_u<0x112, 0xF>(0u, v));
    v = max(v, dpp_u<0x114, 0xF>(0u, v));
    v = max(v, dpp_u<0x118, 0xF>(0u, v));
    v = max(v, dpp_u<0x142, 0xA>(0u, v));
    v = max(v, dpp_u<0x143, 0xC>(0u, v));
    return v;
}

// The key's bits without the mapping of -0 to +0 (so that they turn back into
// the float); norm_key maps them onto the ordering key.
__device__ inline uint32_t raw_key(float f) {
    const uint32_t u = __float_as_uint(f);
    return u ^ (uint32_t(int32_t(u) >> 31) | 0x80000000u);
}
__device__ inline float raw_float(uint32_t k) {
    return __uint_as_float(k ^ (uint32_t(int32_t(~k) >> 31) | 0x80000000u));
}
__device__ inline uint32_t norm_key(uint32_t k) { return k == 0x7fffffffu ? 0x80000000u : k; }
// lanes below this one in a mask
__device__ inline int count_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0));
}

// (start, count) of a heap node over n points: the left child takes
// floor(c / 2) of a node's c points
__device__ inline int2 node_range(int n, int node) {
    const unsigned v = unsigned(node) + 1u;
    const int depth = 31 - __clz(v);
    int start = 0, cnt = n;
    for (int l = depth - 1; l >= 0; --l) {
        const int half = cnt >> 1;
        if ((v >> l) & 1u) {
            start += half;
            cnt -= half;
        } else {
            cnt = half;
        }
    }
    return make_int2(start, cnt);
}

// Set-up of the grid-wide levels in a single launch: ranges of the nodes
// above the workgroup-built subtrees, the error flag and the histograms
// cleared, the box accumulators of every such level initialised.
struct PrepArgs {
    int2 *range;
    int n, n_nodes;
    int *flag;
    int *hist;
    int64_t n_hist;
    uint32_t *boxu;  // [node][2][dp]: lo words all-ones, hi words zero
    int n_box, dp;
};
__global__ void k_prep(const PrepArgs p) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i == 0) *p.flag = 0;
    if (i < p.n_hist) p.hist[i] = 0;
    if (i < p.n_box) p.boxu[i] = ((i / p.dp) & 1) ? 0u : 0xffffffffu;
    if (i < p.n_nodes) p.range[i] = node_range(p.n, int(i));
}

// ---- initial copy: one array per dimension, non-finite check, root box -------
// kInitRows rows at a time: contiguous reads with a fixed dimension per thread
// (so its extent stays in registers), a transposition in LDS (rows padded to
// an odd length), a contiguous write per dimension.
template <int DP>
struct InitCfg {
    static constexpr int rows = DP <= 16 ? 256 : 64;  // a tile
    static constexpr int tiles = 2048 / rows;         // of one block
};
template <int DP>
__global__ __launch_bounds__(kBlock) void k_init(const float *__restrict__ P, int64_t n, int d,
                                                 float *__restrict__ cur, int64_t ns,
                                                 int *__restrict__ idx, int *__restrict__ flag,
                                                 uint32_t *__restrict__ boxu) {
    constexpr int R = InitCfg<DP>::rows, ST = DP + 1;
    constexpr int RB = kBlock / DP;  // rows of one pass of the block
    __shared__ float s[R * ST];
    __shared__ uint32_t sb[2][DP];
    const int t = threadIdx.x, j = t % DP, rg = t / DP;
    if (t < 2 * DP) sb[t / DP][t % DP] = t < DP ? 0xffffffffu : 0u;
    bool bad = false;
    uint32_t lo = ~0u, hi = 0u;
    for (int it = 0; it < InitCfg<DP>::tiles; ++it) {
        const int64_t r0 = (int64_t(blockIdx.x) * InitCfg<DP>::tiles + it) * R;
        if (r0 >= n) break;
        const int rows = int(n - r0 < R ? n - r0 : R);
        __syncthreads();
        if (j < d) {
#pragma unroll
            for (int q = 0; q < R / RB; ++q) {
                const int r = q * RB + rg;
                if (r < rows) {
                    const float v = P[(r0 + r) * d + j];
                    bad |= !isfinite(v);
                    s[r * ST + j] = v;
                    const uint32_t k = f2key(v);
                    lo = min(lo, k);
                    hi = max(hi, k);
                }
            }
        }
        __syncthreads();
        if (t < rows) idx[r0 + t] = int(r0) + t;
        for (int i = t; i < d * R; i += kBlock) {
            const int jj = i / R, r = i % R;
            if (r < rows) cur[jj * ns + r0 + r] = s[r * ST + jj];
        }
    }
    if (bad) atomicOr(flag, 1);
    if (j < d && lo <= hi) {
        atomicMin(&sb[0][j], lo);
        atomicMax(&sb[1][j], hi);
    }
    __syncthreads();
    if (t < d) {
        atomicMin(&boxu[t], sb[0][t]);
        atomicMax(&boxu[DP + t], sb[1][t]);
    }
}

// the other way, for the long rows that k_seg_build reads in place: one array
// per dimension -> rows of DP floats
template <int DP>
__global__ __launch_bounds__(kBlock) void k_rows(const float *__restrict__ cur, int64_t ns, int64_t n,
                                                 int d, float *__restrict__ rows) {
    constexpr int R = 64, ST = DP + 1;
    __shared__ float s[R * ST];
    const int t = threadIdx.x;
    const int64_t r0 = int64_t(blockIdx.x) * R;
    const int cnt = int(n - r0 < R ? n - r0 : R);
    for (int i = t; i < DP * R; i += kBlock) {
        const int j = i / R, r = i % R;
        s[r * ST + j] = j < d && r < cnt ? cur[j * ns + r0 + r] : 0.f;
    }
    __syncthreads();
    for (int i = t; i < cnt * DP; i += kBlock) rows[r0 * DP + i] = s[(i / DP) * ST + i % DP];
}

// ---- grid-wide level: five launches ------------------------------------------
//   A  split dimension and box of each segment from the accumulated box keys,
//      first digit histogram;
//   B  selection step on digit 0, second digit histogram;
//   C  selection step on digit 1, third digit histogram;
//   D  selection step on digit 2 (the median key is known), per-block counts
//      of keys below / equal to it;
//   E  stable partition (each block sums the counts of the blocks before it)
//      with the children's box keys accumulated for the next level.
// A selection step is a block-wide scan of the segment's histogram; every
// block of the segment takes the same step, the first block stores it.
// Digits are up to 11 bits wide, starting below the bits that the whole
// segment shares (the bits above the highest bit where its extremes differ);
// three digits always suffice, and a segment whose median key is known skips
// the remaining histograms.  Histograms are cleared by the kernel after the
// one that reads them.
constexpr int kDigitBits = 11, kBins = 1 << kDigitBits;
__device__ inline int digit_width(int bits) { return bits < kDigitBits ? bits : kDigitBits; }

// block-wide: the selection after one more digit (all threads return it)
__device__ Sel select_step(const int *__restrict__ H, Sel s) {
    __shared__ int wsum[kBlock / 64];
    __shared__ int sbin[2];
    if (s.bits == 0) return s;  // uniform: the same Sel in the whole block
    const int width = digit_width(s.bits), shift = s.bits - width;
    const uint32_t dm = (1u << width) - 1u;
    constexpr int PER = kBins / kBlock;
    static_assert(PER == 8, "two 16-byte loads per thread");
    int c[PER], sum = 0;
    {
        const int4 *h4 = reinterpret_cast<const int4 *>(H + threadIdx.x * PER);
        const int4 x = h4[0], y = h4[1];
        c[0] = x.x, c[1] = x.y, c[2] = x.z, c[3] = x.w;
        c[4] = y.x, c[5] = y.y, c[6] = y.z, c[7] = y.w;
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) sum += c[q];
    // inclusive prefix of the threads' sums: within each wave by shuffles,
    // then the sums of the waves before
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    for (int q = 0; q < wv; ++q) incl += wsum[q];
    const int excl = incl - sum;
    if (excl <= s.rank && s.rank < incl) {
        int rem = s.rank - excl, bin = threadIdx.x * PER;
#pragma unroll
        for (int q = 0; q < PER - 1; ++q) {
            if (rem >= c[q] && bin == threadIdx.x * PER + q) {
                rem -= c[q];
                ++bin;
            }
        }
        sbin[0] = bin;
        sbin[1] = rem;
    }
    __syncthreads();
    Sel r = s;
    r.prefix |= uint32_t(sbin[0]) << shift;
    r.mask |= dm << shift;
    r.rank = sbin[1];
    r.bits = shift;
    __syncthreads();  // wsum / sbin are reused by the next step
    return r;
}

// histogram of the current digit of the keys matching the selection prefix
// (col: the split dimension's array at the segment's start)
template <int CH>
__device__ void hist_digit(const float *__restrict__ col, int e0, int e1, Sel s,
                           int *__restrict__ gh) {
    __shared__ int h[kBins];
    if (s.bits == 0) return;  // uniform
    const int width = digit_width(s.bits), shift = s.bits - width;
    const uint32_t dm = (1u << width) - 1u;
    for (int i = threadIdx.x; i < kBins; i += kBlock) h[i] = 0;
    __syncthreads();
    constexpr int IT = CH / kBlock;
    float v[IT];
#pragma unroll
    for (int q = 0; q < IT; ++q) {
        const int e = e0 + threadIdx.x + q * kBlock;
        v[q] = e < e1 ? col[e] : 0.f;
    }
#pragma unroll
    for (int q = 0; q < IT; ++q) {
        const int e = e0 + threadIdx.x + q * kBlock;
        const uint32_t k = f2key(v[q]);
        if (e < e1 && (k & s.mask) == s.prefix) atomicAdd(&h[(k >> shift) & dm], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kBins; i += kBlock)
        if (h[i]) atomicAdd(&gh[i], h[i]);
}

// this block's share of a segment's histogram bins, cleared
__device__ inline void clear_share(int *__restrict__ gh, int chunk, int bps) {
    const int per = (kBins + bps - 1) / bps;
    const int b0 = chunk * per, b1 = min(kBins, b0 + per);
    for (int i = b0 + threadIdx.x; i < b1; i += kBlock) gh[i] = 0;
}

// A: split dimension, box, first selection state, digit-0 histogram
template <int DP, int CH>
__global__ __launch_bounds__(kBlock) void k_level_a(const float *__restrict__ cur, int64_t ns, int d,
                                                    const int2 *__restrict__ range, int node0,
                                                    int bps, const uint32_t *__restrict__ boxu,
                                                    float *__restrict__ box,
                                                    int *__restrict__ split_dim,
                                                    Sel *__restrict__ sel0,
                                                    int *__restrict__ hist0) {
    const int seg = blockIdx.x / bps, chunk = blockIdx.x % bps;
    const int node = node0 + seg;
    const int2 r = range[node];
    __shared__ uint32_t slo[DP], shi[DP];
    __shared__ int sbest;
    if (threadIdx.x < DP) {
        slo[threadIdx.x] = boxu[(int64_t(node) * 2) * DP + threadIdx.x];
        shi[threadIdx.x] = boxu[(int64_t(node) * 2 + 1) * DP + threadIdx.x];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        // widest extent, lowest dimension on ties
        int best = 0;
        float bestext = -1.0f;
        for (int j = 0; j < d; ++j) {
            const float ext = key2f(shi[j]) - key2f(slo[j]);
            if (ext > bestext) {
                bestext = ext;
                best = j;
            }
        }
        sbest = best;
    }
    __syncthreads();
    const int best = sbest;
    const uint32_t klo = slo[best], khi = shi[best];
    // every key of the segment shares the bits above the highest bit where
    // the extremes differ: the digits start below them
    const uint32_t diff = klo ^ khi;
    const int bits = diff ? 32 - __clz(diff) : 0;
    const uint32_t mask = bits >= 32 ? 0u : ~((1u << bits) - 1u);
    const Sel s0 = Sel{klo & mask, mask, r.y / 2, bits};
    if (chunk == 0) {
        if (threadIdx.x < DP) {
            const int j = threadIdx.x;
            box[int64_t(node) * 2 * DP + j] = j < d ? key2f(slo[j]) : 0.f;
            box[int64_t(node) * 2 * DP + DP + j] = j < d ? key2f(shi[j]) : 0.f;
        }
        if (threadIdx.x == 0) {
            split_dim[node] = best;
            sel0[seg] = s0;
        }
    }
    const int e0 = chunk * CH, e1 = min(r.y, e0 + CH);
    hist_digit<CH>(cur + best * ns + r.x, e0, e1, s0, hist0 + int64_t(seg) * kBins);
}

// B, C: selection step on the previous digit, next digit's histogram (C
// clears the digit-0 histogram)
template <int CH>
__global__ __launch_bounds__(kBlock) void k_level_bc(const float *__restrict__ cur, int64_t ns,
                                                     const int2 *__restrict__ range,
                                                     const int *__restrict__ split_dim, int node0,
                                                     int bps, const Sel *__restrict__ sel_in,
                                                     Sel *__restrict__ sel_out,
                                                     const int *__restrict__ hist_in,
                                                     int *__restrict__ hist_out,
                                                     int *__restrict__ hist_clear) {
    const int seg = blockIdx.x / bps, chunk = blockIdx.x % bps;
    const int2 r = range[node0 + seg];
    const int js = split_dim[node0 + seg];
    const Sel s = select_step(hist_in + int64_t(seg) * kBins, sel_in[seg]);
    if (chunk == 0 && threadIdx.x == 0) sel_out[seg] = s;
    if (hist_clear) clear_share(hist_clear + int64_t(seg) * kBins, chunk, bps);
    const int e0 = chunk * CH, e1 = min(r.y, e0 + CH);
    hist_digit<CH>(cur + js * ns + r.x, e0, e1, s, hist_out + int64_t(seg) * kBins);
}

// D: last selection step; counts of keys below / equal to the median key
template <int CH>
__global__ __launch_bounds__(kBlock) void k_level_count(const float *__restrict__ cur, int64_t ns,
                                                        const int2 *__restrict__ range,
                                                        const int *__restrict__ split_dim,
                                                        int node0, int bps,
                                                        const Sel *__restrict__ sel_in,
                                                        Sel *__restrict__ sel_out,
                                                        const int *__restrict__ hist_in,
                                                        int *__restrict__ hist_clear,
                                                        int2 *__restrict__ counts) {
    const int seg = blockIdx.x / bps, chunk = blockIdx.x % bps;
    const int2 r = range[node0 + seg];
    const float *col = cur + split_dim[node0 + seg] * ns + r.x;
    const int e0 = chunk * CH, e1 = min(r.y, e0 + CH);
    constexpr int IT = CH / kBlock;
    float x[IT];
#pragma unroll
    for (int q = 0; q < IT; ++q) {
        const int e = e0 + threadIdx.x + q * kBlock;
        x[q] = e < e1 ? col[e] : 0.f;
    }
    const Sel s = select_step(hist_in + int64_t(seg) * kBins, sel_in[seg]);
    if (chunk == 0 && threadIdx.x == 0) sel_out[seg] = s;
    clear_share(hist_clear + int64_t(seg) * kBins, chunk, bps);
    const uint32_t v = s.prefix;
    int nl = 0, ne = 0;
#pragma unroll
    for (int q = 0; q < IT; ++q) {
        const int e = e0 + threadIdx.x + q * kBlock;
        const uint32_t key = f2key(x[q]);
        nl += e < e1 && key < v;
        ne += e < e1 && key == v;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        nl += __shfl_xor(nl, off);
        ne += __shfl_xor(ne, off);
    }
    __shared__ int sl[kBlock / 64], se[kBlock / 64];
    if ((threadIdx.x & 63) == 0) {
        sl[threadIdx.x >> 6] = nl;
        se[threadIdx.x >> 6] = ne;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int a = 0, b = 0;
        for (int q = 0; q < kBlock / 64; ++q) {
            a += sl[q];
            b += se[q];
        }
        counts[blockIdx.x] = make_int2(a, b);
    }
}

// E: stable partition; every element's destination first, then one dimension
// after another (reads and the two runs of writes are contiguous), with the
// children's box keys accumulated on the way.  Bound by the moves: 2 (d + 1) n
// x 4 bytes a level.
template <int DP, int CH>
__global__ __launch_bounds__(kBlock) void k_level_scatter(const int *__restrict__ idx_in,
                                                          int *__restrict__ idx_out,
                                                          const float *__restrict__ cur,
                                                          float *__restrict__ nxt, int64_t ns,
                                                          const int2 *__restrict__ range,
                                                          const int *__restrict__ split_dim,
                                                          int node0, int bps,
                                                          const Sel *__restrict__ sel,
                                                          const int2 *__restrict__ counts,
                                                          int *__restrict__ hist_clear,
                                                          int *__restrict__ err, int d,
                                                          uint32_t *__restrict__ boxu_next) {
    const int seg = blockIdx.x / bps, chunk = blockIdx.x % bps;
    const int2 r = range[node0 + seg];
    const int e0 = chunk * CH, e1 = min(r.y, e0 + CH);
    const float *col = cur + split_dim[node0 + seg] * ns + r.x;
    constexpr int IT = CH / kBlock;
    constexpr int NW = kBlock / 64;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    // this thread's elements: e0 + q * kBlock + thread
    float x[IT];
#pragma unroll
    for (int q = 0; q < IT; ++q) {
        const int e = e0 + q * kBlock + threadIdx.x;
        x[q] = e < e1 ? col[e] : 0.f;
    }
    const Sel s = sel[seg];
    const uint32_t v = s.prefix;
    const int req = s.rank;  // equal keys that go left
    const int m = r.y / 2;
    clear_share(hist_clear + int64_t(seg) * kBins, chunk, bps);
    __shared__ int wl[IT][NW], we[IT][NW];
    __shared__ int pl[NW], pe[NW];
    {
        // counts of the segment's blocks before this one
        int a = 0, b = 0;
        for (int c = threadIdx.x; c < chunk; c += kBlock) {
            const int2 q = counts[seg * bps + c];
            a += q.x;
            b += q.y;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            a += __shfl_xor(a, o);
            b += __shfl_xor(b, o);
        }
        if (lane == 0) {
            pl[w] = a;
            pe[w] = b;
        }
    }
    uint64_t bl[IT], be[IT];
#pragma unroll
    for (int q = 0; q < IT; ++q) {
        const bool valid = e0 + q * kBlock + int(threadIdx.x) < e1;
        const uint32_t key = f2key(x[q]);
        bl[q] = __ballot(valid && key < v);
        be[q] = __ballot(valid && key == v);
        if (lane == 0) {
            wl[q][w] = __popcll(bl[q]);
            we[q][w] = __popcll(be[q]);
        }
    }
    __syncthreads();
    int run_l = 0, run_e = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        run_l += pl[q];
        run_e += pe[q];
    }
    int pos[IT];
    uint32_t left = 0;  // bit q: element q goes left
#pragma unroll
    for (int q = 0; q < IT; ++q) {
        int ol = run_l, oe = run_e;
#pragma unroll
        for (int u = 0; u < NW; ++u) {
            if (u < w) {
                ol += wl[q][u];
                oe += we[q][u];
            }
            run_l += wl[q][u];
            run_e += we[q][u];
        }
        const int e = e0 + q * kBlock + threadIdx.x;
        const bool less = (bl[q] >> lane) & 1, eq = (be[q] >> lane) & 1;
        const int less_before = ol + __popcll(bl[q] & lanemask_lt());
        const int eq_before = oe + __popcll(be[q] & lanemask_lt());
        const bool lf = less || (eq && eq_before < req);
        const int left_before = less_before + min(eq_before, req);
        int p = lf ? left_before : m + (e - left_before);
        if (e < e1 && (p < 0 || p >= r.y)) {  // cannot happen for a correct select
            atomicOr(err, 2);
            p = min(max(p, 0), r.y - 1);
        }
        pos[q] = r.x + p;
        left |= (lf ? 1u : 0u) << q;
    }
#pragma unroll
    for (int q = 0; q < IT; ++q) {
        const int e = e0 + q * kBlock + threadIdx.x;
        if (e < e1) idx_out[pos[q]] = idx_in[r.x + e];
    }
    __shared__ uint32_t sb[4][DP];  // left lo, left hi, right lo, right hi
    if (threadIdx.x < 4 * DP)
        sb[threadIdx.x / DP][threadIdx.x % DP] = ((threadIdx.x / DP) & 1) ? 0u : 0xffffffffu;
    __syncthreads();
    constexpr int JB = 4;  // dimensions whose loads are in flight together
    for (int j0 = 0; j0 < d; j0 += JB) {
        float y[JB][IT];
#pragma unroll
        for (int b = 0; b < JB; ++b) {
            const float *src = cur + min(j0 + b, d - 1) * ns + r.x;
#pragma unroll
            for (int q = 0; q < IT; ++q) {
                const int e = e0 + q * kBlock + threadIdx.x;
                y[b][q] = src[min(e, r.y - 1)];
            }
        }
#pragma unroll
        for (int b = 0; b < JB; ++b) {
            const int j = j0 + b;
            if (j >= d) break;  // uniform
            float *dst = nxt + j * ns;
            uint32_t ll = ~0u, lh = 0u, rl = ~0u, rh = 0u;
#pragma unroll
            for (int q = 0; q < IT; ++q) {
                const int e = e0 + q * kBlock + threadIdx.x;
                if (e < e1) {
                    dst[pos[q]] = y[b][q];
                    const uint32_t k = f2key(y[b][q]);
                    const bool lf = (left >> q) & 1;
                    ll = min(ll, lf ? k : ~0u);
                    lh = max(lh, lf ? k : 0u);
                    rl = min(rl, lf ? ~0u : k);
                    rh = max(rh, lf ? 0u : k);
                }
            }
            if (!boxu_next) continue;  // uniform
            ll = wave_umin(ll);
            lh = wave_umax(lh);
            rl = wave_umin(rl);
            rh = wave_umax(rh);
            if (lane == 63) {
                if (ll <= lh) {
                    atomicMin(&sb[0][j], ll);
                    atomicMax(&sb[1][j], lh);
                }
                if (rl <= rh) {
                    atomicMin(&sb[2][j], rl);
                    atomicMax(&sb[3][j], rh);
                }
            }
        }
    }
    if (!boxu_next) return;  // uniform
    __syncthreads();
    // the children of a node are adjacent: [2 node + 1][lo, hi], [2 node + 2]..
    uint32_t *out = boxu_next + int64_t(2 * (node0 + seg) + 1) * 2 * DP;
    if (threadIdx.x < 4 * DP) {
        const int c = threadIdx.x / DP, j = threadIdx.x % DP;
        if (j < d && sb[c & 2][j] <= sb[(c & 2) + 1][j]) {
            if (c & 1)
                atomicMax(&out[c * DP + j], sb[c][j]);
            else
                atomicMin(&out[c * DP + j], sb[c][j]);
        }
    }
}

__device__ inline float round_up_f(double x) {
    x *= 1.0 + 0x1p-46;  // covers the FP64 evaluation error
    float f = (float)x;
    if ((double)f < x) f = nextafterf(f, __builtin_inff());
    return f;
}

// ---- internal nodes: lambda <= max_c (|C - C_c| + lambda_c), and <= the
//      distance from C to the farthest box corner ------------------------------
// corner: that distance; dc[c]: |C - C_c| (-1 for an empty child)
template <int DP>
__device__ void lambda_parts(bool empty0, bool empty1, int node, int d, const float *__restrict__ box,
                             double &corner, double (&dc)[2]) {
    const float *b = box + int64_t(node) * 2 * DP;
    const float *cb = box + int64_t(2 * node + 1) * 2 * DP;  // both children
    double s = 0.0, s0 = 0.0, s1 = 0.0;
#pragma unroll 4
    for (int j = 0; j < d; ++j) {
        const float c = 0.5f * (b[j] + b[DP + j]);
        const double h = fmax((double)b[DP + j] - c, (double)c - b[j]);
        s += h * h;
        const double d0 = (double)c - (double)(0.5f * (cb[j] + cb[DP + j]));
        const double d1 = (double)c - (double)(0.5f * (cb[2 * DP + j] + cb[3 * DP + j]));
        s0 += d0 * d0;
        s1 += d1 * d1;
    }
    corner = sqrt(s);
    dc[0] = empty0 ? -1.0 : sqrt(s0);
    dc[1] = empty1 ? -1.0 : sqrt(s1);
}
__device__ inline float lambda_of(double corner, const double (&dc)[2], float lam0, float lam1) {
    double via = 0.0;
    if (dc[0] >= 0.0) via = fmax(via, dc[0] + (double)lam0);
    if (dc[1] >= 0.0) via = fmax(via, dc[1] + (double)lam1);
    return round_up_f(fmin(corner, via));
}

// ---- one workgroup builds a segment's subtree ------------------------------------
// Levels l0 .. l1 - 1 of the segment under node seg of level l0.  sidx holds
// local row numbers in the current order (two buffers).  While a level has
// fewer nodes than waves, several waves share a node: a histogram of 256
// equal steps between the node's extremes finds the step that holds the
// median (equal steps spread the LDS atomics, where leading key bits crowd
// into a few bins), and the few keys of that step are bisected with ballots,
// ending once a single one is left; a step with more than 512 keys goes
// through 8-bit digits instead.  Then a node of up to 512 points is one wave's
// work, its keys in registers.
//
// l1 == L: the tree's leaves are written (points, leaf blocks, permutation,
// boxes, lambda), then the subtree's internal lambda.  l1 < L: the partition
// so far goes to `nxt` / `idx_out`, for a second launch of more and smaller
// workgroups.
//
// What bounds it: instruction issue (about 150 instructions per 64 points and
// level) where the segments fill the chip, the chain of dependent steps where
// they do not.  All-kNN of 10,000 points in d = 3 (both launches 42 us): the
// call 303 -> 215 us against five launches a level down to 1024 points and
// one launch each for leaves, leaf blocks and lambda.  4M x 1M, d = 16: 17.7 ->
// 15.75 ms (one array per dimension in the grid-wide levels: the key passes
// read 4 of 64 bytes a point, and no pass over the points for the boxes).
constexpr int kSegLds = 159 * 1024;
constexpr int kSmallSeg = 1024;  // points of a segment that four waves finish
template <int DP, int NW>
struct SegCfg {
    static constexpr int waves = NW;
    static constexpr bool staged = DP <= 16;  // points in LDS
    // 16 rows of a leaf at a time per wave, for the long rows
    static constexpr int tile_rows = 16, tile_row = DP + 1;
    static constexpr size_t fixed = size_t(NW) * 256 * 4                        // histograms
                                    + size_t(NW) * 2 * DP * 4                   // box parts
                                    + 64 * 4 * 2 + 256                          // counts, misc
                                    + size_t(NW) * 256 * 4                      // the median step's keys
                                    + (staged ? 0 : size_t(NW) * (tile_rows * tile_row + DP) * 4);
    // most points of a segment: a wave's node has at most 512 points
    static int most(int d) {
        const int lanes = NW * 496;
        if (!staged) return lanes;
        const int m = int((kSegLds - fixed - 64) / (size_t(d) * 4 + 4)) & ~31;
        return m < lanes ? m : lanes;
    }
    static size_t bytes(int d, int cap) {
        return fixed + (staged ? size_t(cap) * d * 4 : 0) + size_t(cap) * 4;
    }
};
// waves of the workgroup that splits a segment down to kSmallSeg points.  Up to
// 16 dimensions 16 waves reach 7936 points in LDS where 8 reach 3968 (us with 16 and
// with 8, d = 3: 5000 points 137 and 167, 1.5M 720 and 740; 2000 points, where
// one level fewer is shared, 110 and 102).  Longer rows are read in place, and
// there 16 waves gain up to 100,000 points (d = 32: 5000 points 241 and 336,
// 100,000 596 and 621) and lose 2% at 400,000 (d = 24: 948 and 930).
constexpr int mid_waves(int DP) { return DP <= 16 ? 16 : 8; }
constexpr int kEndWaves = 4;  // of the one that finishes it

struct SegArgs {
    const float *rows;     // rows of `stride` floats (the input, or long rows), or NULL
    int stride, check;     // check: the rows are the input, not seen by a launch before
    const float *cur;      // else one array of ns floats per dimension
    const int *idx_in;     // original rows (NULL: identity)
    float *nxt;            // l1 < L: the partitioned points (arrays; rows of DP floats where
    int *idx_out;          // they are long) and original rows
    int64_t ns;
    int n, d, l0, l1, L, cap;
    int2 *range;
    float *box, *lam;
    int *split_dim, *err;
    float *pts, *lpts;
    int *perm;
    int leaf_slots;
    int own_flag;          // this launch writes the error flag (no grid-wide levels ran)
};

__device__ inline void wave_lds_sync() {
    // LDS writes of this wave visible to its other lanes; no workgroup wait
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

template <int DP, int NW>
__global__ __launch_bounds__(64 * NW) void k_seg_build(const SegArgs a) {
    using C = SegCfg<DP, NW>;
    constexpr int NT = 64 * NW;
    constexpr bool kStaged = C::staged;
    constexpr int NG = 64 / DP;
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const int seg = blockIdx.x, d = a.d, cap = a.cap;
    const int2 rr = node_range(a.n, (1 << a.l0) - 1 + seg);
    const int base = uni(rr.x), c = uni(rr.y);
    // (start, count) of the sub-th node `levels` levels below the segment
    auto sub_range = [&](int levels, int sub) -> int2 {
        int start = base, cnt = c;
        for (int l = levels - 1; l >= 0; --l) {
            const int half = cnt >> 1;
            const bool right = (sub >> l) & 1;
            start += right ? half : 0;
            cnt = right ? cnt - half : half;
        }
        return make_int2(start, cnt);
    };

    extern __shared__ __align__(16) char smem[];
    int *s_hist = reinterpret_cast<int *>(smem);                          // [NW][256]
    uint32_t *s_box = reinterpret_cast<uint32_t *>(s_hist + NW * 256);    // [NW][2][DP]
    int *s_cnt = reinterpret_cast<int *>(s_box + NW * 2 * DP);            // [2][64]
    int *s_misc = s_cnt + 128;                                            // [64]
    uint32_t *s_list = reinterpret_cast<uint32_t *>(s_misc + 64);         // [NW / 2][512]
    float *s_tile = reinterpret_cast<float *>(s_list + NW * 256);         // long rows only
    uint32_t *s_pts =  // [d][cap] raw keys
        reinterpret_cast<uint32_t *>(s_tile + (kStaged ? 0 : NW * (C::tile_rows * C::tile_row + DP)));
    uint16_t *s_idx = reinterpret_cast<uint16_t *>(s_pts + (kStaged ? d * cap : 0));  // [2][cap]

    if (tid < 8) s_misc[tid] = 0;
    __syncthreads();
    // stage the points; the input rows are checked here when no launch before
    // this one has seen them
    const int j_l = lane % DP, grp = lane / DP;
    bool bad = false;
    if (a.rows) {
        if (kStaged || a.check) {
            const float *p = a.rows + int64_t(base) * a.stride;
            if (j_l < d) {
#pragma unroll 4
                for (int e = wave * NG + grp; e < c; e += NW * NG) {
                    const float v = p[int64_t(e) * a.stride + j_l];
                    bad |= !isfinite(v);
                    if constexpr (kStaged) s_pts[j_l * cap + e] = raw_key(v);
                }
            }
        }
    } else if constexpr (kStaged) {
        for (int j = 0; j < d; ++j) {
#pragma unroll 8
            for (int e = tid; e < c; e += NT) s_pts[j * cap + e] = raw_key(a.cur[j * a.ns + base + e]);
        }
    }
    if (bad && a.check) atomicOr(&s_misc[0], 1);
    auto raw = [&](int row, int j) -> uint32_t {
        if constexpr (kStaged)
            return s_pts[j * cap + row];
        else
            return raw_key(a.rows[int64_t(base + row) * a.stride + j]);
    };
    auto X = [&](int row, int j) -> float {
        if constexpr (kStaged)
            return raw_float(s_pts[j * cap + row]);
        else
            return a.rows[int64_t(base + row) * a.stride + j];
    };
    for (int e = tid; e < c; e += NT) s_idx[e] = uint16_t(e);
    __syncthreads();

    // Box keys of the elements whose rows a wave's lanes hold (a lane without an
    // element repeats one of the node): lane j gets dimension j.  Short rows:
    // a lane per element; longer ones: a lane per dimension over elements e0 ..
    // e1 - 1 of src.
    auto node_box = [&](auto &row, const uint16_t *src, int e0, int e1, uint32_t &lo,
                        uint32_t &hi) __attribute__((always_inline)) {
        constexpr int R = sizeof(row) / sizeof(row[0]);
        lo = ~0u;
        hi = 0u;
        if constexpr (DP <= 8) {
#pragma unroll
            for (int j = 0; j < DP; ++j) {
                if (j < d) {  // uniform
                    uint32_t l = ~0u, h = 0u;
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const uint32_t k = raw(row[q], j);
                        l = min(l, k);
                        h = max(h, k);
                    }
                    l = (uint32_t)__builtin_amdgcn_readlane((int)wave_umin(l), 63);
                    h = (uint32_t)__builtin_amdgcn_readlane((int)wave_umax(h), 63);
                    lo = lane == j ? l : lo;
                    hi = lane == j ? h : hi;
                }
            }
        } else {
            if (j_l < d) {
#pragma unroll 4
                for (int e = e0 + grp; e < e1; e += NG) {
                    const uint32_t k = raw(src[e], j_l);
                    lo = min(lo, k);
                    hi = max(hi, k);
                }
            }
#pragma unroll
            for (int off = DP; off < 64; off <<= 1) {
                lo = min(lo, (uint32_t)__shfl_xor((int)lo, off));
                hi = max(hi, (uint32_t)__shfl_xor((int)hi, off));
            }
        }
        lo = norm_key(lo);
        hi = norm_key(hi);
    };
    // widest dimension (lowest on ties) from lane j's keys of dimension j;
    // writes the box when asked
    auto choose = [&](int node, uint32_t lo, uint32_t hi, bool write) __attribute__((always_inline)) -> int {
        const float flo = lane < d ? key2f(lo) : 0.f, fhi = lane < d ? key2f(hi) : 0.f;
        const float ext = lane < d ? fhi - flo : -1.0f;
        if (write && lane < DP) {
            a.box[int64_t(node) * 2 * DP + lane] = flo;
            a.box[int64_t(node) * 2 * DP + DP + lane] = fhi;
        }
        float mx = ext;
#pragma unroll
        for (int off = DP > 32 ? 32 : DP / 2; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
        mx = __int_as_float(uni(__float_as_int(mx)));
        const uint64_t cand = __ballot(lane < d && ext == mx);
        const int js = cand ? __builtin_ctzll(cand) : 0;
        if (write && lane == 0) a.split_dim[node] = js;
        return js;
    };
    // The key at rank `rank` among n keys in registers (unused ones ~0), whose
    // bits above `top` are those of `prefix`: a range [vlo, vhi] that holds it
    // and no key that differs from it; rank becomes the rank within the range.
    auto bisect = [&](auto &key, int n, uint32_t prefix, uint32_t top, int &rank, uint32_t &vlo,
                      uint32_t &vhi) __attribute__((always_inline)) {
        constexpr int R = sizeof(key) / sizeof(key[0]);
        int below = 0, upto = n;  // keys below the range, and up to its end
        uint32_t last = top ? (top << 1) - 1u : 0u;  // bits not yet fixed
#pragma unroll 1
        for (uint32_t bit = top; bit && upto - below > 1; bit >>= 1) {
            const uint32_t t = prefix | bit;
            int cnt = 0;
#pragma unroll
            for (int q = 0; q < R; ++q) cnt += __popcll(__ballot(key[q] < t));
            const bool high = cnt <= rank;
            prefix = high ? t : prefix;
            below = high ? cnt : below;
            upto = high ? upto : cnt;
            last = bit - 1u;
        }
        vlo = prefix;
        vhi = prefix | last;
        rank -= below;
    };
    // which of this wave's elements (in use: e0 + 64 q + lane < e1) have keys
    // below vlo, and in [vlo, vhi]
    auto compare = [&](auto &key, int e0, int e1, uint32_t vlo, uint32_t vhi, auto &bl, auto &be, int &nl,
                       int &ne) __attribute__((always_inline)) {
        constexpr int R = sizeof(key) / sizeof(key[0]);
        nl = ne = 0;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const uint64_t on = __ballot(e0 + 64 * q + lane < e1);
            bl[q] = __ballot(key[q] < vlo) & on;
            be[q] = __ballot(key[q] >= vlo && key[q] <= vhi) & on;
            nl += __popcll(bl[q]);
            ne += __popcll(be[q]);
        }
    };
    // stable partition of them: the keys below vlo and the first `rank` of
    // those in [vlo, vhi] go left (run_l, run_e: how many of both the waves
    // before have)
    auto place = [&](auto &row, uint16_t *dst, int e0, int e1, auto &bl, auto &be, int run_l, int run_e,
                     int rank, int cc) __attribute__((always_inline)) {
        constexpr int R = sizeof(row) / sizeof(row[0]);
        bool off = false;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int e = e0 + 64 * q + lane;
            const int eq_before = run_e + count_below(be[q]);
            const int left_before = run_l + count_below(bl[q]) + min(eq_before, rank);
            const bool eq = __builtin_amdgcn_inverse_ballot_w64(be[q]);
            const bool left = __builtin_amdgcn_inverse_ballot_w64(bl[q]) || (eq && eq_before < rank);
            const uint32_t pos = uint32_t(left ? left_before : cc / 2 + (e - left_before));
            const bool valid = e < e1;
            off |= valid && pos >= uint32_t(cc);  // cannot happen for a correct select
            if (valid) dst[min(pos, uint32_t(cc - 1))] = row[q];
            run_l += __popcll(bl[q]);
            run_e += __popcll(be[q]);
        }
        if (off) atomicOr(&s_misc[0], 2);
    };
    // one node of up to 64 R points, this wave's work
    auto wave_node = [&](auto r_const, int node, int cc, const uint16_t *src, uint16_t *dst) __attribute__((always_inline)) {
        constexpr int R = decltype(r_const)::value;
        uint16_t row[R];
#pragma unroll
        for (int q = 0; q < R; ++q) row[q] = src[min(q * 64 + lane, cc - 1)];
        uint32_t lo, hi;
        node_box(row, src, 0, cc, lo, hi);
        const int js = choose(node, lo, hi, true);
        const uint32_t klo = (uint32_t)__builtin_amdgcn_readlane((int)lo, js);
        const uint32_t khi = (uint32_t)__builtin_amdgcn_readlane((int)hi, js);
        uint32_t key[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const uint32_t k = norm_key(raw(row[q], js));
            key[q] = q * 64 + lane < cc ? k : ~0u;
        }
        const uint32_t top = klo != khi ? 0x80000000u >> __clz(klo ^ khi) : 0u;
        const uint32_t prefix = top ? klo & ~((top << 1) - 1u) : klo;
        int rank = cc / 2, nl, ne;
        uint32_t vlo, vhi;
        bisect(key, cc, prefix, top, rank, vlo, vhi);
        uint64_t bl[R], be[R];
        compare(key, 0, cc, vlo, vhi, bl, be, nl, ne);
        place(row, dst, 0, cc, bl, be, 0, 0, rank, cc);
    };

    int cb = 0;
    for (int lv = a.l0; lv < a.l1; ++lv) {
        const int nsub = 1 << (lv - a.l0);
        const int node0 = (1 << lv) - 1 + seg * nsub;
        const uint16_t *src0 = s_idx + cb * cap;
        uint16_t *dst0 = s_idx + (cb ^ 1) * cap;
        const int most = (c + nsub - 1) / nsub;
        if (most <= 512 && (nsub * 2 >= NW || most <= 256)) {
            for (int sub = wave; sub < nsub; sub += NW) {
                const int2 nr = sub_range(lv - a.l0, sub);
                const int o = uni(nr.x) - base, cc = uni(nr.y);
                if (lane == 0) a.range[node0 + sub] = nr;
                const uint16_t *src = src0 + o;
                uint16_t *dst = dst0 + o;
                if (most <= 64)
                    wave_node(std::integral_constant<int, 1>{}, node0 + sub, cc, src, dst);
                else if (most <= 128)
                    wave_node(std::integral_constant<int, 2>{}, node0 + sub, cc, src, dst);
                else if (most <= 256)
                    wave_node(std::integral_constant<int, 4>{}, node0 + sub, cc, src, dst);
                else
                    wave_node(std::integral_constant<int, 8>{}, node0 + sub, cc, src, dst);
            }
        } else {
            // gw waves share a node, all nodes of the level at once.  Every
            // group takes the same barriers.
            constexpr int R = 8;
            const int gw = max(1, NW >> (lv - a.l0));
            const int sub = wave / gw, gi = wave % gw, g0 = wave - gi;
            const int node = node0 + sub;  // (nsub = NW / gw: every wave has one)
            const int2 nr = sub_range(lv - a.l0, sub);
            const int o = uni(nr.x) - base, cc = uni(nr.y);
            const uint16_t *src = src0 + o;
            uint16_t *dst = dst0 + o;
            // this wave's share of the elements, a contiguous range
            const int share = ((cc + gw - 1) / gw + 63) & ~63;
            const int b0 = min(cc, gi * share), b1 = min(cc, b0 + share);
            uint16_t row[R];
#pragma unroll
            for (int q = 0; q < R; ++q) row[q] = src[min(b0 + q * 64 + lane, cc - 1)];
            uint32_t lo, hi;
            node_box(row, src, b0, b1, lo, hi);
            if (lane < DP) {
                s_box[(wave * 2) * DP + lane] = lo;
                s_box[(wave * 2 + 1) * DP + lane] = hi;
            }
            int *hist = s_hist + g0 * 256;
            uint32_t *list = s_list + sub * 512;
            for (int i = gi * 64 + lane; i < 256; i += gw * 64) hist[i] = 0;
            if (gi == 0 && lane == 0) s_cnt[64 + g0] = 0;
            __syncthreads();
#pragma unroll 1
            for (int q = 0; q < gw; ++q) {
                if (lane < DP) {
                    lo = min(lo, s_box[((g0 + q) * 2) * DP + lane]);
                    hi = max(hi, s_box[((g0 + q) * 2 + 1) * DP + lane]);
                }
            }
            const int js = choose(node, lo, hi, gi == 0);
            if (gi == 0 && lane == 0) a.range[node] = nr;
            const uint32_t klo = (uint32_t)__builtin_amdgcn_readlane((int)lo, js);
            const uint32_t khi = (uint32_t)__builtin_amdgcn_readlane((int)hi, js);
            const uint32_t diff = klo ^ khi;
            const uint32_t top = diff ? 0x80000000u >> __clz(diff) : 0u;
            const uint32_t common = diff ? klo & ~((top << 1) - 1u) : klo;
            const float flo = key2f(klo), fext = key2f(khi) - flo;
            const float step = fminf(256.0f / fext, 3.402823466e38f);  // (0 when the extent overflows)
            // monotone in the key: both roundings are
            auto bin_of = [&](uint32_t k) __attribute__((always_inline)) -> int {
                return int(fminf((key2f(k) - flo) * step, 255.0f));
            };
            uint32_t key[R];
            int bins[R];
#pragma unroll
            for (int q = 0; q < R; ++q) {
                key[q] = norm_key(raw(row[q], js));
                bins[q] = bin_of(key[q]);
                if (diff && b0 + q * 64 + lane < b1) atomicAdd(&hist[bins[q]], 1);
            }
            __syncthreads();
            // the bin of histogram h that holds rank, the rank within it, its count
            auto locate = [&](int &rank, int &in) __attribute__((always_inline)) -> int {
                const int4 h = reinterpret_cast<const int4 *>(hist)[lane];
                const int sum = h.x + h.y + h.z + h.w;
                int incl = sum;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const int t = __shfl_up(incl, off);
                    if (lane >= off) incl += t;
                }
                const int excl = incl - sum;
                const uint64_t who = __ballot(excl <= rank && rank < incl);
                const int owner = who ? __builtin_ctzll(who) : 0;
                int rem = rank - __builtin_amdgcn_readlane(excl, owner);
                const int h0 = __builtin_amdgcn_readlane(h.x, owner);
                const int h1 = __builtin_amdgcn_readlane(h.y, owner);
                const int h2 = __builtin_amdgcn_readlane(h.z, owner);
                int bin = owner * 4;
                in = h0;
                if (rem >= in) {
                    rem -= in;
                    ++bin;
                    in = h1;
                    if (rem >= in) {
                        rem -= in;
                        ++bin;
                        in = h2;
                        if (rem >= in) {
                            rem -= in;
                            ++bin;
                            in = __builtin_amdgcn_readlane(h.w, owner);
                        }
                    }
                }
                rank = rem;
                return bin;
            };
            const int m = cc / 2;
            int rank = m, in = 0, bin = 0;
            if (diff) bin = locate(rank, in);
            const bool few = in <= 512;
            if (diff && few) {
#pragma unroll
                for (int q = 0; q < R; ++q)
                    if (bins[q] == bin && b0 + q * 64 + lane < b1) list[atomicAdd(&s_cnt[64 + g0], 1)] = key[q];
            }
            // (a flag per parity of the level; this barrier is also the list's)
            if (diff && !few && lane == 0) s_misc[4 + (lv & 1)] = 1;
            __syncthreads();
            const bool digits = s_misc[4 + (lv & 1)] != 0;
            if (tid == 0) s_misc[4 + ((lv + 1) & 1)] = 0;
            uint32_t vlo = klo, vhi = klo;
            if (diff && few) {
                uint32_t lk[R];
#pragma unroll
                for (int q = 0; q < R; ++q) lk[q] = q * 64 + lane < in ? list[q * 64 + lane] : ~0u;
                bisect(lk, in, common, top, rank, vlo, vhi);
                // the range is one key's among the list's only: that key itself
                uint32_t v = vlo;
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const uint64_t at = __ballot(q * 64 + lane < in && lk[q] >= vlo && lk[q] <= vhi);
                    if (at) v = (uint32_t)__builtin_amdgcn_readlane((int)lk[q], __builtin_ctzll(at));
                }
                vlo = vhi = v;
            }
            if (digits) {
                // 8-bit digits below the common prefix, for the groups that
                // need them
                const bool mine = diff != 0 && !few;
                int bits = mine ? 32 - __clz(diff) : 0;
                uint32_t prefix = common;
                if (mine) rank = m;
#pragma unroll 1
                for (int it = 0; it < 4; ++it) {  // at most 32 bits
                    __syncthreads();
                    const int width = bits < 8 ? bits : 8, shift = bits - width;
                    const uint32_t dm = (1u << width) - 1u;
                    if (bits > 0)
                        for (int i = gi * 64 + lane; i < 256; i += gw * 64) hist[i] = 0;
                    __syncthreads();
                    if (bits > 0) {
                        const uint32_t mask = bits >= 32 ? 0u : ~((1u << bits) - 1u);
#pragma unroll
                        for (int q = 0; q < R; ++q)
                            if (b0 + q * 64 + lane < b1 && (key[q] & mask) == prefix)
                                atomicAdd(&hist[(key[q] >> shift) & dm], 1);
                    }
                    __syncthreads();
                    if (bits > 0) {
                        prefix |= uint32_t(locate(rank, in)) << shift;
                        bits = shift;
                    }
                }
                if (mine) vlo = vhi = prefix;
            }
            // stable partition: counts of this wave's range, then places
            int nl, ne;
            uint64_t bl[R], be[R];
            compare(key, b0, b1, vlo, vhi, bl, be, nl, ne);
            if (lane == 0) {
                s_cnt[wave] = nl;
                s_cnt[32 + wave] = ne;
            }
            __syncthreads();
            int run_l = 0, run_e = 0;
            for (int q = 0; q < gi; ++q) {
                run_l += s_cnt[g0 + q];
                run_e += s_cnt[32 + g0 + q];
            }
            place(row, dst, b0, b1, bl, be, run_l, run_e, rank, cc);
        }
        __syncthreads();  // the next level reads every node's partition
        cb ^= 1;
    }
    const uint16_t *fin = s_idx + cb * cap;
    if (a.own_flag) {
        if (tid == 0) *a.err = s_misc[0];
    } else if (tid == 0 && s_misc[0]) {
        atomicOr(a.err, s_misc[0]);
    }
    auto orig = [&](int row) { return a.idx_in ? a.idx_in[base + row] : base + row; };

    if (a.l1 < a.L) {  // hand the partition to the next launch
        for (int e = tid; e < c; e += NT) a.idx_out[base + e] = orig(fin[e]);
        if constexpr (kStaged) {
            for (int j = 0; j < d; ++j)
                for (int e = tid; e < c; e += NT) a.nxt[j * a.ns + base + e] = X(fin[e], j);
        } else {
            for (int e = wave * NG + grp; e < c; e += NW * NG)
                a.nxt[int64_t(base + e) * DP + j_l] = j_l < d ? X(fin[e], j_l) : 0.f;
        }
        return;
    }

    // ---- leaves: points in tree order, leaf block, box, exact lambda ---------
    const int first_leaf = (1 << a.L) - 1;
    const int nleaf = 1 << (a.L - a.l0);
    const int leaf0 = seg * nleaf;
    // the subtree's lambda in LDS (heap order within the subtree) while the
    // chain of levels runs, and the parts that need only the boxes
    float *s_lam = reinterpret_cast<float *>(s_list);
    double *s_part = reinterpret_cast<double *>(s_hist);
    const bool chain = (2 * nleaf - 1) * 4 <= NW * 1024 && (nleaf - 1) * 24 <= NW * 1024;
    for (int s = wave; s < nleaf; s += NW) {
        const int leaf = leaf0 + s, node = first_leaf + leaf;
        const int2 nr = sub_range(a.L - a.l0, s);
        const int o = uni(nr.x) - base, cc = uni(nr.y);
        float *lp = a.lpts + int64_t(leaf) * a.leaf_slots * DP;
        float lo = __builtin_inff(), hi = -__builtin_inff();  // lane j: dimension j
        double s2 = -1.0;
        if constexpr (DP <= 16) {
            // lane = row
            const int row = lane < cc ? fin[o + lane] : 0;
            float x[DP];
#pragma unroll
            for (int j = 0; j < DP; ++j) x[j] = lane < cc && j < d ? X(row, j) : 0.f;
            if (lane < cc) {
                a.perm[nr.x + lane] = orig(row);
#pragma unroll
                for (int j = 0; j < DP; j += 4)
                    *reinterpret_cast<float4 *>(a.pts + int64_t(nr.x + lane) * DP + j) =
                        make_float4(x[j], x[j + 1], x[j + 2], x[j + 3]);
            }
            if (lane < a.leaf_slots) {
                const float pad = 3.402823466e38f;
#pragma unroll
                for (int j = 0; j < DP; j += 4)
                    *reinterpret_cast<float4 *>(lp + lane * DP + j) =
                        lane < cc ? make_float4(x[j], x[j + 1], x[j + 2], x[j + 3])
                                  : make_float4(pad, pad, pad, pad);
            }
            if (lane < cc) s2 = 0.0;
#pragma unroll
            for (int j = 0; j < DP; ++j) {
                if (j < d) {
                    const uint32_t k = raw_key(x[j]);
                    const float l = raw_float(norm_key((uint32_t)__builtin_amdgcn_readlane(
                        (int)wave_umin(lane < cc ? k : ~0u), 63)));
                    const float h = raw_float(norm_key((uint32_t)__builtin_amdgcn_readlane(
                        (int)wave_umax(lane < cc ? k : 0u), 63)));
                    if (cc > 0 && lane == j) {
                        lo = l;
                        hi = h;
                    }
                    const double df = (double)x[j] - (double)(0.5f * (l + h));
                    if (lane < cc) s2 = fma(df, df, s2);
                }
            }
        } else {
            // a few rows at a time through this wave's LDS tile: whole rows
            // are read and written, lane j takes dimension j's extent; a second
            // pass, a lane per row, takes lambda
            constexpr int TR = C::tile_rows;
            float *tile = s_tile + wave * (TR * C::tile_row + DP);
            float *cen = tile + TR * C::tile_row;
            const int row = lane < cc ? fin[o + lane] : 0;
            if (lane < cc) a.perm[nr.x + lane] = orig(row);
            auto fill = [&](int r0) {  // rows r0 .. r0 + TR - 1
                wave_lds_sync();
#pragma unroll
                for (int r = grp; r < TR; r += NG) {
                    const int rw = __shfl(row, min(r0 + r, 63));
                    tile[r * C::tile_row + j_l] = r0 + r < cc && j_l < d ? X(rw, j_l) : 0.f;
                }
                wave_lds_sync();
            };
            for (int r0 = 0; r0 < a.leaf_slots; r0 += TR) {
                fill(r0);
                for (int r = 0; r < TR && r0 + r < a.leaf_slots; ++r) {
                    const bool on = r0 + r < cc;
                    if (lane < DP) {
                        const float v = on ? tile[r * C::tile_row + lane] : 3.402823466e38f;
                        lp[(r0 + r) * DP + lane] = v;
                        if (on) {
                            a.pts[int64_t(nr.x + r0 + r) * DP + lane] = v;
                            const float z = v == 0.0f ? 0.0f : v;
                            lo = fminf(lo, z);
                            hi = fmaxf(hi, z);
                        }
                    }
                }
            }
            if (lane < DP) cen[lane] = lane < d ? 0.5f * (lo + hi) : 0.f;
            for (int r0 = 0; r0 < cc; r0 += TR) {
                fill(r0);
                if (lane >= r0 && lane < r0 + TR && lane < cc) {
                    s2 = 0.0;
                    for (int j = 0; j < d; ++j) {
                        const double df = (double)tile[(lane - r0) * C::tile_row + j] - (double)cen[j];
                        s2 = fma(df, df, s2);
                    }
                }
            }
        }
        // largest s2 (non-negative doubles order as their bits): the high words
        // first, then the low words of the lanes that hold the largest
        const uint64_t sb = s2 >= 0.0 ? uint64_t(__double_as_longlong(s2)) : 0u;
        const uint32_t sh = (uint32_t)__builtin_amdgcn_readlane((int)wave_umax(uint32_t(sb >> 32)), 63);
        const uint32_t sl = (uint32_t)__builtin_amdgcn_readlane(
            (int)wave_umax(uint32_t(sb >> 32) == sh ? uint32_t(sb) : 0u), 63);
        s2 = __longlong_as_double((long long)((uint64_t(sh) << 32) | sl));
        const float lam = cc > 0 ? round_up_f(sqrt(s2)) : 0.f;
        if (lane < DP) {
            a.box[int64_t(node) * 2 * DP + lane] = lane < d ? lo : 0.f;
            a.box[int64_t(node) * 2 * DP + DP + lane] = lane < d ? hi : 0.f;
        }
        if (lane == 0) {
            a.range[node] = nr;
            a.split_dim[node] = -1;
            a.lam[node] = lam;
            if (chain) s_lam[nleaf - 1 + s] = lam;
        }
    }
    // the rows past the last point (tile loops may read them)
    if (seg == int(gridDim.x) - 1)
        for (int i = tid; i < kPadRows * DP; i += NT) a.pts[int64_t(a.n) * DP + i] = 0.f;
    __syncthreads();
    // the subtree's internal lambda, bottom up
    if (chain) {
        for (int i = tid; i < nleaf - 1; i += NT) {
            const int lv = 31 - __clz(i + 1), sub = i + 1 - (1 << lv);
            const int nc = sub_range(lv, sub).y;
            double corner, dc[2];
            lambda_parts<DP>(nc / 2 == 0, nc - nc / 2 == 0, (((1 << a.l0) + seg) << lv) - 1 + sub, d, a.box,
                             corner, dc);
            s_part[3 * i] = corner;
            s_part[3 * i + 1] = dc[0];
            s_part[3 * i + 2] = dc[1];
        }
        for (int lv = a.L - a.l0 - 1; lv >= 0; --lv) {
            __syncthreads();
            for (int sub = tid; sub < (1 << lv); sub += NT) {
                const int i = (1 << lv) - 1 + sub;
                const double dc[2] = {s_part[3 * i + 1], s_part[3 * i + 2]};
                const float v = lambda_of(s_part[3 * i], dc, s_lam[2 * i + 1], s_lam[2 * i + 2]);
                s_lam[i] = v;
                a.lam[(((1 << a.l0) + seg) << lv) - 1 + sub] = v;
            }
        }
        return;
    }
    for (int lv = a.L - 1; lv >= a.l0; --lv) {
        const int cnt = 1 << (lv - a.l0);
        for (int i = tid; i < cnt; i += NT) {
            const int node = (1 << lv) - 1 + seg * cnt + i;
            const int nc = sub_range(lv - a.l0, i).y;
            double corner, dc[2];
            lambda_parts<DP>(nc / 2 == 0, nc - nc / 2 == 0, node, d, a.box, corner, dc);
            a.lam[node] = lambda_of(corner, dc, a.lam[2 * node + 1], a.lam[2 * node + 2]);
        }
        __syncthreads();
    }
}

// levels [0, top - 1] in one block, bottom up.  The parts that need only the
// boxes come first (every node at once, kept in LDS kTopNodes at a time from
// the bottom levels on); the chain of levels then only adds and compares.
constexpr int kTopNodes = 4096;
template <int DP>
__global__ __launch_bounds__(1024) void k_lambda_top(int n, int top, int d,
                                                     const float *__restrict__ box,
                                                     float *__restrict__ lam) {
    __shared__ double part[3][kTopNodes];
    for (int hi = top; hi > 0;) {
        // levels lo .. hi - 1 have at most kTopNodes nodes
        int lo = hi - 1;
        while (lo > 0 && (1 << hi) - (1 << (lo - 1)) <= kTopNodes) --lo;
        const bool fits = (1 << hi) - (1 << lo) <= kTopNodes;
        const int first = (1 << lo) - 1, cnt = (1 << hi) - (1 << lo);
        if (fits) {
            __syncthreads();
            for (int i = threadIdx.x; i < cnt; i += blockDim.x) {
                const int nc = node_range(n, first + i).y;
                double corner, dc[2];
                lambda_parts<DP>(nc / 2 == 0, nc - nc / 2 == 0, first + i, d, box, corner, dc);
                part[0][i] = corner;
                part[1][i] = dc[0];
                part[2][i] = dc[1];
            }
        }
        for (int lv = hi - 1; lv >= lo; --lv) {
            __syncthreads();
            for (int i = threadIdx.x; i < (1 << lv); i += blockDim.x) {
                const int node = (1 << lv) - 1 + i;
                double corner, dc[2];
                if (fits) {
                    corner = part[0][node - first];
                    dc[0] = part[1][node - first];
                    dc[1] = part[2][node - first];
                } else {
                    const int nc = node_range(n, node).y;
                    lambda_parts<DP>(nc / 2 == 0, nc - nc / 2 == 0, node, d, box, corner, dc);
                }
                lam[node] = lambda_of(corner, dc, lam[2 * node + 1], lam[2 * node + 2]);
            }
        }
        hi = lo;
    }
}

// The kernel's dynamic LDS limit, a property of the function on a device that
// all builds share: set once, to the most that any build asks for.  (Set per
// launch to that launch's size, a smaller build of another thread could lower
// it between a larger one's call and its launch.)
template <int DP, int NW>
hipError_t raise_lds_limit() {
    static std::atomic<uint64_t> done{0};  // one bit per device
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev >= 0 && dev < 64 ? uint64_t(1) << dev : 0u;
    if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_seg_build<DP, NW>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kSegLds);
    if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
    return e;
}

template <int DP>
knn_status build_impl(const float *points, int64_t n, int d, int leaf, hipStream_t s,
                      knn_tree *t, int *flag, hipEvent_t done) {
    using Mid = SegCfg<DP, mid_waves(DP)>;
    using End = SegCfg<DP, kEndWaves>;
    const int L = t->depth;
    const int nn = int(n);
    int *idxA = nullptr, *idxB = nullptr, *hist = nullptr;
    uint32_t *boxu = nullptr;
    float *cur = nullptr, *nxt = nullptr;
    Sel *sel = nullptr;
    int2 *counts = nullptr;
    struct Guard {
        hipStream_t s;
        std::vector<void *> p;
        ~Guard() {
            dev_free_many(p.data(), int(p.size()), s);
        }
    } g{s, {}};
    auto get = [&](auto **ptr, size_t cnt) -> hipError_t {
        hipError_t e = alloc_async(ptr, cnt, s);
        if (e == hipSuccess) g.p.push_back(*ptr);
        return e;
    };
    const int64_t ns = (n + 63) & ~int64_t(63);

    auto cmax = [&](int lv) { return int((n + (int64_t(1) << lv) - 1) >> lv); };
    constexpr int CH = kHistChunk, CM = kMoveChunk;
    // grid-wide levels down to what one workgroup splits, that workgroup's
    // levels down to what four waves finish
    const int mid_most = Mid::most(d);
    const int end_most = std::min({kSmallSeg, End::most(d), mid_most});
    int n_global = 0, maxseg = 1, maxblk = 1;
    for (int q = 0; q < L && cmax(q) > mid_most; ++q) {
        n_global = q + 1;
        maxseg = std::max(maxseg, 1 << q);
        maxblk = std::max(maxblk, (1 << q) * ((cmax(q) + CM - 1) / CM));
    }
    int l_mid = n_global;
    while (l_mid < L && cmax(l_mid) > end_most) ++l_mid;
    const bool two = l_mid > n_global;
    if (n_global > 0 || two) {
        KNN_HIP(get(&idxA, n));
        KNN_HIP(get(&cur, size_t(ns) * DP));
    }
    if (n_global > 0) {
        KNN_HIP(get(&idxB, n));
        KNN_HIP(get(&nxt, size_t(ns) * DP));
        KNN_HIP(get(&boxu, size_t(2 << n_global) * 2 * DP));
        KNN_HIP(get(&sel, 4 * size_t(maxseg)));
        KNN_HIP(get(&hist, 3 * size_t(maxseg) * kBins));
        KNN_HIP(get(&counts, size_t(maxblk)));
        PrepArgs p{};
        p.range = t->range;
        p.n = nn;
        p.n_nodes = (1 << n_global) - 1;
        p.flag = flag;
        p.hist = hist;
        p.n_hist = 3 * int64_t(maxseg) * kBins;
        p.boxu = boxu;
        p.n_box = int((size_t(2) << n_global) * 2 * DP);
        p.dp = DP;
        const int64_t tot = std::max<int64_t>({p.n_hist, int64_t(p.n_box), int64_t(p.n_nodes)});
        k_prep<<<int((tot + 255) / 256), 256, 0, s>>>(p);
        const int64_t rows = int64_t(InitCfg<DP>::rows) * InitCfg<DP>::tiles;
        k_init<DP><<<int((n + rows - 1) / rows), kBlock, 0, s>>>(points, n, d, cur, ns, idxA, flag, boxu);
    }
    int *H[3] = {hist, hist + size_t(maxseg) * kBins, hist + 2 * size_t(maxseg) * kBins};
    Sel *S[4] = {sel, sel + maxseg, sel + 2 * maxseg, sel + 3 * maxseg};
    for (int l = 0; l < n_global; ++l) {
        const int nseg = 1 << l, node0 = nseg - 1;
        const int bps = (cmax(l) + CH - 1) / CH;
        const int nblk = nseg * bps;
        const int bpm = (cmax(l) + CM - 1) / CM, nblm = nseg * bpm;
        k_level_a<DP, CH><<<nblk, kBlock, 0, s>>>(cur, ns, d, t->range, node0, bps, boxu, t->box,
                                                  t->split_dim, S[0], H[0]);
        k_level_bc<CH><<<nblk, kBlock, 0, s>>>(cur, ns, t->range, t->split_dim, node0, bps, S[0], S[1],
                                               H[0], H[1], nullptr);
        k_level_bc<CH><<<nblk, kBlock, 0, s>>>(cur, ns, t->range, t->split_dim, node0, bps, S[1], S[2],
                                               H[1], H[2], H[0]);
        k_level_count<CM><<<nblm, kBlock, 0, s>>>(cur, ns, t->range, t->split_dim, node0, bpm, S[2],
                                                  S[3], H[2], H[1], counts);
        k_level_scatter<DP, CM><<<nblm, kBlock, 0, s>>>(idxA, idxB, cur, nxt, ns, t->range, t->split_dim,
                                                        node0, bpm, S[3], counts, H[2], flag, d,
                                                        l + 1 < n_global ? boxu : nullptr);
        std::swap(idxA, idxB);
        std::swap(cur, nxt);
    }
    SegArgs a{};
    if (n_global == 0) {
        a.rows = points;
        a.stride = d;
    } else if (!Mid::staged) {
        k_rows<DP><<<int((n + 63) / 64), kBlock, 0, s>>>(cur, ns, n, d, nxt);
        std::swap(cur, nxt);
        a.rows = cur;
        a.stride = DP;
    }
    a.check = n_global == 0;
    a.cur = cur;
    a.idx_in = n_global > 0 ? idxA : nullptr;
    a.ns = ns;
    a.n = nn;
    a.d = d;
    a.L = L;
    a.range = t->range;
    a.box = t->box;
    a.lam = t->lam;
    a.split_dim = t->split_dim;
    a.err = flag;
    a.pts = t->pts;
    a.lpts = t->lpts;
    a.perm = t->perm;
    a.leaf_slots = t->leaf_slots;
    auto launch = [&](auto cfg, auto kernel, int waves, int l0, int l1) -> hipError_t {
        a.l0 = l0;
        a.l1 = l1;
        a.cap = (cmax(l0) + 31) & ~31;
        const size_t lds = decltype(cfg)::bytes(d, a.cap);
        if (lds > size_t(kSegLds)) return hipErrorInvalidValue;
        hipError_t e = raise_lds_limit<DP, decltype(cfg)::waves>();
        if (e != hipSuccess) return e;
        kernel<<<1 << l0, 64 * waves, lds, s>>>(a);
        return hipGetLastError();
    };
    if (two) {
        a.nxt = n_global > 0 ? nxt : cur;
        a.idx_out = n_global > 0 ? idxB : idxA;
        a.own_flag = n_global == 0;
        KNN_HIP(launch(Mid{}, &k_seg_build<DP, mid_waves(DP)>, mid_waves(DP), n_global, l_mid));
        a.cur = a.nxt;
        a.rows = Mid::staged ? nullptr : a.nxt;
        a.stride = DP;
        a.check = 0;
        a.idx_in = a.idx_out;
    }
    a.own_flag = n_global == 0 && !two;
    // (few segments: more waves shorten each one's chain, the chip has room)
    if ((1 << l_mid) <= 256)
        KNN_HIP(launch(Mid{}, &k_seg_build<DP, mid_waves(DP)>, mid_waves(DP), l_mid, L));
    else
        KNN_HIP(launch(End{}, &k_seg_build<DP, kEndWaves>, kEndWaves, l_mid, L));
    if (l_mid > 0) k_lambda_top<DP><<<1, 1024, 0, s>>>(nn, l_mid, d, t->box, t->lam);
    KNN_HIP(hipGetLastError());
    KNN_HIP(hipEventRecord(done, s));
    return KNN_OK;
}

}  // namespace

void free_tree(knn_tree *t) {
    if (!t) return;
    int cur = 0;
    const bool switch_dev = hipGetDevice(&cur) == hipSuccess && cur != t->device;
    if (switch_dev) (void)hipSetDevice(t->device);
    void *blocks[] = {t->pts, t->lpts, t->perm, t->range, t->box, t->lam, t->split_dim};
    dev_free_many(blocks, 7, t->stream);
    if (switch_dev) (void)hipSetDevice(cur);
    delete t;
}

namespace {

// one build in flight: its tree, stream, error flag and timing events
struct BuildJob {
    knn_tree *t = nullptr;
    hipStream_t s = nullptr;
    int *flag = nullptr;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
};

void drop_job(BuildJob &job) {
    free_async(job.flag, job.s);
    if (job.ev0) (void)hipEventDestroy(job.ev0);
    if (job.ev1) (void)hipEventDestroy(job.ev1);
    free_tree(job.t);
    job = BuildJob{};
}

// allocations and every launch of one build on stream s; no host wait
knn_status build_enqueue(const float *points, int64_t n, int d, int leaf, hipStream_t s,
                         BuildJob &job) {
    knn_tree *t = new knn_tree();
    job.t = t;
    job.s = s;
    t->n = n;
    t->d = d;
    t->dp = pad_dim(d);
    t->leaf_size = leaf;
    t->depth = depth_for(n, leaf);
    t->n_nodes = (int64_t(2) << t->depth) - 1;
    t->n_leaves = int64_t(1) << t->depth;
    t->first_leaf = t->n_leaves - 1;
    {
        const int64_t max_leaf = (n + t->n_leaves - 1) / t->n_leaves;
        t->leaf_slots = int32_t((max_leaf + 7) / 8 * 8);
    }
    t->stream = s;
    const int dp = t->dp;
    hipError_t e = hipGetDevice(&t->device);
    e = e ? e : alloc_async(&t->pts, size_t(n + kPadRows) * dp, s);
    e = e ? e : alloc_async(&t->lpts, size_t(t->n_leaves) * t->leaf_slots * dp, s);
    e = e ? e : alloc_async(&t->perm, size_t(n), s);
    e = e ? e : alloc_async(&t->range, size_t(t->n_nodes), s);
    e = e ? e : alloc_async(&t->box, size_t(t->n_nodes) * 2 * dp, s);
    e = e ? e : alloc_async(&t->lam, size_t(t->n_nodes), s);
    e = e ? e : alloc_async(&t->split_dim, size_t(t->n_nodes), s);
    e = e ? e : alloc_async(&job.flag, 1, s);
    if (e != hipSuccess) {
        drop_job(job);
        return fail(e == hipErrorOutOfMemory ? KNN_E_OOM : KNN_E_DEVICE,
                    std::string("knn_build_tree: allocation failed: ") + hipGetErrorString(e));
    }
    e = hipEventCreate(&job.ev0);
    e = e ? e : hipEventCreate(&job.ev1);
    e = e ? e : hipEventRecord(job.ev0, s);
    if (e != hipSuccess) {
        drop_job(job);
        return hip_fail(e, "knn_build_tree: set-up", __FILE__, __LINE__);
    }
    knn_status st;
    switch (dp) {
        case 4: st = build_impl<4>(points, n, d, leaf, s, t, job.flag, job.ev1); break;
        case 8: st = build_impl<8>(points, n, d, leaf, s, t, job.flag, job.ev1); break;
        case 16: st = build_impl<16>(points, n, d, leaf, s, t, job.flag, job.ev1); break;
        case 32: st = build_impl<32>(points, n, d, leaf, s, t, job.flag, job.ev1); break;
        default: st = build_impl<64>(points, n, d, leaf, s, t, job.flag, job.ev1); break;
    }
    if (st != KNN_OK) {
        (void)hipStreamSynchronize(s);  // the launches already queued must end first
        drop_job(job);
    }
    return st;
}

// wait for a build, check its flag; the tree is handed out or freed
knn_status build_finish(BuildJob &job, knn_tree **out) {
    int hflag = 0;
    hipError_t e = hipMemcpyAsync(&hflag, job.flag, sizeof(int), hipMemcpyDeviceToHost, job.s);
    e = e ? e : hipStreamSynchronize(job.s);
    if (e != hipSuccess) {
        drop_job(job);
        return hip_fail(e, "knn_build_tree: device work", __FILE__, __LINE__);
    }
    if (hflag & 1) {
        drop_job(job);
        return fail(KNN_E_NONFINITE, "knn_build_tree: non-finite coordinate in input");
    }
    if (hflag & 2) {
        drop_job(job);
        return fail(KNN_E_DEVICE, "knn_build_tree: internal partition inconsistency");
    }
    (void)hipEventElapsedTime(&job.t->ms_build, job.ev0, job.ev1);
    free_async(job.flag, job.s);
    (void)hipEventDestroy(job.ev0);
    (void)hipEventDestroy(job.ev1);
    *out = job.t;
    job = BuildJob{};
    return KNN_OK;
}

// A helper thread that issues the second build of a pair.  It lives for the
// whole process (never joined: it waits for work on a condition variable),
// so a pair build costs no thread start.  One pair build uses it at a time;
// a concurrent caller starts a thread of its own.
class BuildHelper {
  public:
    static BuildHelper &get() {
        static BuildHelper *h = new BuildHelper();  // never destroyed
        return *h;
    }
    std::mutex use;  // held by the pair build that owns the helper
    void run(std::function<void()> f) {
        std::lock_guard<std::mutex> lock(mu_);
        task_ = std::move(f);
        pending_ = true;
        cv_.notify_all();
    }
    void wait() {
        std::unique_lock<std::mutex> lock(mu_);
        cv_.wait(lock, [&] { return !pending_; });
    }

  private:
    BuildHelper() { std::thread([this] { loop(); }).detach(); }
    void loop() {
        for (;;) {
            std::function<void()> f;
            {
                std::unique_lock<std::mutex> lock(mu_);
                cv_.wait(lock, [&] { return pending_; });
                f = std::move(task_);
            }
            f();
            std::lock_guard<std::mutex> lock(mu_);
            pending_ = false;
            cv_.notify_all();
        }
    }
    std::mutex mu_;
    std::condition_variable cv_;
    std::function<void()> task_;
    bool pending_ = false;
};

// a second stream per device (default priority) for the pair build
hipError_t aux_stream(hipStream_t *out) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static hipStream_t streams[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!streams[dev]) {
        e = hipStreamCreateWithFlags(&streams[dev], hipStreamNonBlocking);
        if (e != hipSuccess) return e;
    }
    *out = streams[dev];
    return hipSuccess;
}

}  // namespace

knn_status build_tree(const float *points, int64_t n, int d, int leaf, hipStream_t s,
                      knn_tree **out) {
    BuildJob job;
    KNN_TRY(build_enqueue(points, n, d, leaf, s, job));
    return build_finish(job, out);
}

namespace {

// enqueues the builds of a and (when pb is not NULL) b, b on the second
// stream from the helper thread; on error nothing is left queued or held
knn_status pair_enqueue(const float *pa, int64_t na, const float *pb, int64_t nb, int d, int leaf,
                        hipStream_t s, BuildJob &ja, BuildJob &jb) {
    if (!pb) return build_enqueue(pa, na, d, leaf, s, ja);
    hipStream_t s2;
    KNN_HIP(aux_stream(&s2));
    // the second build may only start once the caller's stream has produced
    // its inputs
    hipEvent_t ready;
    KNN_HIP(hipEventCreateWithFlags(&ready, hipEventDisableTiming));
    hipError_t e = hipEventRecord(ready, s);
    e = e ? e : hipStreamWaitEvent(s2, ready, 0);
    (void)hipEventDestroy(ready);
    if (e != hipSuccess) return hip_fail(e, "knn_build_tree_pair: stream join", __FILE__, __LINE__);
    // the launches of one build take about as long to issue as to run, so
    // the second build is issued from a second host thread
    int dev = 0;
    KNN_HIP(hipGetDevice(&dev));
    knn_status sb = KNN_OK;
    std::string msg_b;
    auto second = [&] {
        if (hipSetDevice(dev) != hipSuccess) {
            sb = KNN_E_DEVICE;
            msg_b = "knn_build_tree_pair: hipSetDevice failed in the build thread";
            return;
        }
        sb = build_enqueue(pb, nb, d, leaf, s2, jb);
        if (sb != KNN_OK) msg_b = get_error();
    };
    BuildHelper &helper = BuildHelper::get();
    std::unique_lock<std::mutex> owner(helper.use, std::try_to_lock);
    std::thread own;
    if (owner.owns_lock())
        helper.run(second);
    else
        own = std::thread(second);
    const knn_status sa = build_enqueue(pa, na, d, leaf, s, ja);
    const std::string msg_a = get_error();
    if (owner.owns_lock())
        helper.wait();
    else
        own.join();
    if (sa != KNN_OK || sb != KNN_OK) {
        knn_tree *tmp = nullptr;
        if (sa == KNN_OK && build_finish(ja, &tmp) == KNN_OK) free_tree(tmp);
        tmp = nullptr;
        if (sb == KNN_OK && build_finish(jb, &tmp) == KNN_OK) free_tree(tmp);
        return sa != KNN_OK ? fail(sa, msg_a) : fail(sb, msg_b);
    }
    return KNN_OK;
}

// waits for both builds; on error neither tree is returned
knn_status pair_finish(BuildJob &ja, BuildJob &jb, hipStream_t s, knn_tree **ta, knn_tree **tb) {
    const bool two = jb.t != nullptr;
    knn_tree *a = nullptr, *b = nullptr;
    const knn_status sa = build_finish(ja, &a);
    const std::string msg_a = get_error();
    const knn_status sb = two ? build_finish(jb, &b) : KNN_OK;
    if (sa != KNN_OK || sb != KNN_OK) {
        if (a) free_tree(a);
        if (b) free_tree(b);
        return sa != KNN_OK ? fail(sa, msg_a) : sb;
    }
    // both builds have completed (finish waited for each stream); the second
    // tree belongs to the caller's stream from now on
    if (b) b->stream = s;
    *ta = a;
    if (tb) *tb = b;
    return KNN_OK;
}

}  // namespace

knn_status build_tree_pair(const float *pa, int64_t na, const float *pb, int64_t nb, int d,
                           int leaf, hipStream_t s, knn_tree **out_a, knn_tree **out_b) {
    BuildJob ja, jb;
    KNN_TRY(pair_enqueue(pa, na, pb, nb, d, leaf, s, ja, jb));
    return pair_finish(ja, jb, s, out_a, out_b);
}

knn_status all_knn(const float *ref_points, int64_t n_ref, const float *query_points,
                   int64_t n_query, int d, int leaf, int k, const knn_opts *opts,
                   int64_t *idx_out, float *dist_out, hipStream_t s) {
    BuildJob ja, jb;
    KNN_TRY(pair_enqueue(ref_points, n_ref, query_points, n_query, d, leaf, s, ja, jb));
    // the search reads the query tree built on the second stream
    hipError_t e = jb.t ? hipStreamWaitEvent(s, jb.ev1, 0) : hipSuccess;
    knn_status st = e == hipSuccess
                        ? search(ja.t, jb.t, k, opts, idx_out, dist_out, s)
                        : hip_fail(e, "knn_all_knn: stream join", __FILE__, __LINE__);
    const std::string msg = get_error();
    knn_tree *ta = nullptr, *tb = nullptr;
    const knn_status sf = pair_finish(ja, jb, s, &ta, &tb);  // input checks of the builds
    if (sf != KNN_OK) return sf;
    if (st == KNN_OK && opts && opts->stats) {
        opts->stats->ms_ref_build = ta->ms_build;
        opts->stats->ms_query_build = tb ? tb->ms_build : 0.f;
    }
    free_tree(ta);
    if (tb) free_tree(tb);
    return st == KNN_OK ? KNN_OK : fail(st, msg);
}

}  // namespace knnx
