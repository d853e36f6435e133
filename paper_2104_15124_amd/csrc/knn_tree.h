// Exact k-NN selection over curve-ordered matrix-core tiles, pruned by a tree
// of projected boxes (gfx950).
//
// The samples are laid out in the Morton order of their principal projections,
// refined by median splits inside groups of 4096 tiles (spatial_mfma.hip), so
// 32 consecutive positions form a compact tile and 64 consecutive tiles (or
// tree nodes) form a compact node of the level above. One wavefront (a
// workgroup of its own) owns one tile of 32 queries. Its scan has two passes.
//
// Pass 1 finds every query's threshold without keeping any candidate. Lane l
// of the matrix-core tile holds the scores of candidate l of each half's 16
// queries, and keeps the D smallest scores it has seen per query, sorted, in
// registers: D median-of-three instructions per query and tile. A query's
// threshold is a value that at least kp of those 32 D scores do not exceed, found
// by bisection (a lane's count, added over the half's lanes); it is at or
// above the query's kp-th score, and close to it while no lane holds more than
// D of the kp nearest: D is 5 up to kp = 96, 8 up to 224, 12 beyond (the mean per
// lane is kp / 32; eight at kp = 256 put 474 candidates below the threshold). The
// tiles are visited as a walk down the tree: a node's (up to 64) children are bounded
// at once, one per lane, against the query tile's box, the pending child with the
// smallest bound is taken first (so the thresholds fall early), and every child is
// re-tested against the wavefront's largest distance threshold when taken. Tiles
// in which some score is at or below its query's threshold are noted; pass 1 ends
// with the walk or when a set number of tiles are noted.
//
// Pass 2 goes over the noted tiles, forms the same scores again and writes
// those at or below the threshold straight into the query's list in global
// scratch: some kp keys per query, each written once. Where the notes were full
// before the walk was over it then goes on with the walk, each tile scored once, its
// keys written in the same way (walking the tree again from its root took
// samples none of whose tiles can be skipped twice the products: Gaussian, n = 100k,
// m = 16 and 64, 22.0 and 35.6 ms against 15.1 and 21.4; 5-manifold, n = 1M, 126 to
// 98). Where the tiles within reach are many (tree_wide_min), the wavefronts end after
// pass 1 and hand their query tiles over to scans that keep no scores: 10.5 and 16.9 ms.
// A list without room for a tile's keys is cut by a lower threshold that at least kp
// of its keys do not exceed. Lists of kp within 32 of their capacity are sorted instead
// once full, and take further keys from a buffer in LDS, 32 at a time (k + margin =
// 256, n = 20k, m = 12: 4.1 ms against 17.4 by a sort per tile and 5.1 by one pass of
// sorted lists; 5-manifold n = 100k 13.6, 35.1 and 19.8). At the end each list is sorted once.
//
// A scan that keeps sorted lists while its thresholds fall appends each query's
// candidates several times over and merges its list some ten times; those
// merges and appends were two thirds of its time. A wavefront whose box held a
// few outlying samples walked for most of a launch (141 of 176 ms on the 8M
// mixture) until boxes were also tested against the single queries (PointTest).
// Whole k-NN calls, before (sorted lists, box tests only) and now: mixture m = 16,
// n = 8M, FP32 144 -> 97 ms, n = 1M BF16 19.9 -> 13.3; 5-manifold m = 64, n = 1M
// 254 -> 97; lifted 3-sphere m = 128, n = 4M, k = 128: 192 -> 103.
//
// Short contractions (SHORT) keep the query fragments and two tiles ahead of
// the products in registers. Long ones keep the query operand in LDS, and first
// bound each tile by the same kind of product over the 8 projected coordinates
// (two BF16 matrix instructions, operands formed from the 32-byte rows of
// projections): a box of 32 samples of a curved 5-manifold lets 2340 of 31250
// tiles through per query tile at n = 1M, the pairwise bound 480 of them,
// 163 hold a neighbour. Only tiles with a pair within reach load their operand
// (1 KB per K-step) and take the full product.
//
// A tile is skipped only when a rigorous bound on its distances exceeds the
// thresholds at that time, which bound the final ones. A threshold counts
// computed scores, a bound speaks of true distances: a counted candidate may lie
// beyond the distance of its threshold by the score's error E_q, so pass 2 tests the
// noted tiles against the threshold and E_q. Should a list end short of kp keys
// all the same, its last score is no bound; its threshold is one: every candidate
// missing from a list has a score above the threshold or a true distance beyond it,
// and the certificate (derivation in knn_mfma.hip) takes the smaller of the two.
//
// The contraction lengths are compiled in four files (knn_tree_*.hip), which
// takes a quarter of the time; knn_tree.hip picks the launcher.
#pragma once

#include <algorithm>
#include <type_traits>

#include "knn_mfma_common.h"

namespace kvb {

namespace {

constexpr int TNQ = 32;      // queries per wavefront
constexpr int TASK = 128;    // noted tiles at which a query tile is handed over
constexpr int TREACH = WAVE * WAVE;   // the reach where every sampled tile is within reach of every sampled query tile
// Tiles in flight. Short contractions stream the fragments of two tiles ahead
// of the products (a tile with no hits is too short to cover the next one's
// loads); long ones the projections of two.
constexpr int TREE_DEPTH = 3;
constexpr int TBUF = 32;     // keys buffered per query of a full list
constexpr float TINF = __builtin_inff();

// the wavefront's LDS state; NOTES: the tiles that pass 1 notes
template <int NOTES>
struct alignas(16) TreeLds {
    float tau[TNQ];                     // score thresholds (-inf: no query)
    float zt[TNQ];                      // thresholds of the projected scores (long contractions)
    float gt[TNQ];                      // thresholds of the squared projected distances
    float yq[TNQ];                      // |y_q|^2
    float box[2 * PR_DIMS];             // the query tile's box
    float gbox[WAVE][2 * PR_DIMS];      // the boxes of the current group of tiles
    float bnd[TREE_LEVELS - 1][WAVE];   // walk: bounds of the pending children of level l >= 1 in row l - 1
    uint64_t mask[TREE_LEVELS];         //       pending children
    int base[TREE_LEVELS];              //       first child
    int lvl;                            //       level of the current pending list
    uint32_t rec[NOTES + TREE_DEPTH];    // the noted tiles, then those in flight when the notes were full
};

// the tree's shape
struct TreeShape {
    int top;
    int cnt[TREE_LEVELS];
    int off[TREE_LEVELS];
};

// The lane of `m` holding the smallest bound (bounds are >= 0, so their bits
// order like unsigned integers; the low 6 bits carry the lane, which breaks
// ties towards the lower lane and costs a relative 2^-17 of resolution).
__device__ __forceinline__ int nearest_lane(uint64_t m, float bound)
{
    const int lane = lane_id();
    uint32_t key = ((m >> lane) & 1ull) ? ((__float_as_uint(bound) & ~63u) | static_cast<uint32_t>(lane)) : ~0u;
    // rotations within rows of 16 lanes, then the rows
    key = min(key, static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(key, 0x128, 0xF, 0xF, true)));
    key = min(key, static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(key, 0x124, 0xF, 0xF, true)));
    key = min(key, static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(key, 0x122, 0xF, 0xF, true)));
    key = min(key, static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(key, 0x121, 0xF, 0xF, true)));
    const auto r16 = __builtin_amdgcn_permlane16_swap(key, key, false, false);
    const uint32_t a16 = r16[0], b16 = r16[1];
    key = min(a16, b16);
    const auto r32 = __builtin_amdgcn_permlane32_swap(key, key, false, false);
    const uint32_t a32 = r32[0], b32 = r32[1];
    key = min(a32, b32);
    return static_cast<int>(__builtin_amdgcn_readfirstlane(key) & 63u);
}

__device__ __forceinline__ const float* node_box(const float* tbox, const float* tree, const TreeShape* sh, int level,
                                                 int v)
{
    return level == 0 ? tbox + static_cast<size_t>(v) * 2 * PR_DIMS
                      : tree + (static_cast<size_t>(sh->off[level]) + v) * 2 * PR_DIMS;
}

__device__ __forceinline__ void load_box(const float* box, float (&b)[2 * PR_DIMS])
{
    const float4* src = reinterpret_cast<const float4*>(box);
#pragma unroll
    for (int u = 0; u < PR_DIMS / 2; ++u) {
        const float4 t = src[u];
        b[4 * u] = t.x;
        b[4 * u + 1] = t.y;
        b[4 * u + 2] = t.z;
        b[4 * u + 3] = t.w;
    }
}

// A group of up to 64 tiles (level 0), one per lane: first tile, pending
// tiles and each lane's tile bound. base < 0: the walk is over.
struct TileGroup {
    uint64_t mask;
    int base;
    float bnd;
};

// Bounds of the children first .. first + 63 of level `level` to the query box
// (the tiles of the fill range [f0, f0 + nfill) are left out). The tiles' boxes
// (level 0) are left in gbox.
__device__ __forceinline__ float child_bound(const float* tbox, const float* tree, const TreeShape* sh, int level,
                                            int first, const float* qbox, BoxBound bb, int f0, int nfill,
                                            float (*gbox)[2 * PR_DIMS], bool& take)
{
    const int lane = lane_id();
    const int v = first + lane;
    take = lane < min(TREE_FAN, sh->cnt[level] - first);
    if (level == 0) take = take && (v < f0 || v >= f0 + nfill);
    if (!take) return __builtin_nanf("");
    float b[2 * PR_DIMS];
    load_box(node_box(tbox, tree, sh, level, v), b);
    if (level == 0) {
#pragma unroll
        for (int u = 0; u < PR_DIMS / 2; ++u)
            reinterpret_cast<float4*>(gbox[lane])[u] = make_float4(b[4 * u], b[4 * u + 1], b[4 * u + 2], b[4 * u + 3]);
    }
    return box_bound(b, qbox, qbox + PR_DIMS, bb);
}

// This lane's query (l31) and half of its projected coordinates, and its
// threshold: a box within reach of the query box may still hold nothing within
// reach of any single query (the corners between them; a tile of outlying
// samples whose box spans a whole region, which alone kept one wavefront
// walking for 141 of 176 ms on the 8M mixture).
struct PointTest {
    float z[PR_DIMS / 2];
    float gt;
    // whether some query lies within its threshold of the box; lo, hi: this
    // lane's half of the box's corners
    __device__ __forceinline__ bool reach(const float4 lo, const float4 hi) const
    {
        const float l[4] = {lo.x, lo.y, lo.z, lo.w}, h[4] = {hi.x, hi.y, hi.z, hi.w};
        float g2 = 0.f;
#pragma unroll
        for (int c = 0; c < PR_DIMS / 2; ++c) {
            const float g = fmaxf(fmaxf(l[c] - z[c], z[c] - h[c]), 0.f);
            g2 = fmaf(g, g, g2);
        }
        g2 += shfl_xor_f32(g2, 32);
        return __ballot(g2 <= gt) != 0ull;
    }
};

// The next group of tiles within reach of thr, after the current one is
// exhausted: up the levels until a pending child within reach, the nearest
// one taken, then down to its tiles. Whole wavefront.
template <int NOTES>
__device__ __forceinline__ TileGroup climb(TreeLds<NOTES>& W, const TreeShape* sh, const float* tbox, const float* tree,
                                        BoxBound bb, const PointTest& pt, float thr, int f0, int nfill)
{
    const int lane = lane_id();
    int lvl = W.lvl;
    if (lvl == 0) {
        if (sh->top == 0) return {0ull, -1, 0.f};
        lvl = 1;
    }
    while (true) {
        const float bl = W.bnd[lvl - 1][lane];
        const uint64_t m = W.mask[lvl] & __ballot(bl <= thr);
        if (!m) {
            if (lvl == sh->top) {
                W.lvl = lvl;
                return {0ull, -1, 0.f};
            }
            ++lvl;
            continue;
        }
        const int c = nearest_lane(m, bl);
        const int node = W.base[lvl] + c;
        const int first = node * TREE_FAN;
        wave_lds_sync();
        if (lane == 0) W.mask[lvl] = m & ~(1ull << c);
        const float4* nb = reinterpret_cast<const float4*>(node_box(tbox, tree, sh, lvl, node));
        const bool in = pt.reach(nb[lane >> 5], nb[PR_DIMS / 4 + (lane >> 5)]);
        wave_lds_sync();
        if (!in) continue;
        bool take;
        float qb[2 * PR_DIMS];
#pragma unroll
        for (int c2 = 0; c2 < 2 * PR_DIMS; ++c2) qb[c2] = W.box[c2];
        const float b = child_bound(tbox, tree, sh, lvl - 1, first, qb, bb, f0, nfill, W.gbox, take);
        const uint64_t mt = __ballot(take);
        --lvl;
        if (lvl == 0) {
            wave_lds_sync();
            if (lane == 0) W.lvl = 0;
            wave_lds_sync();
            return {mt, first, b};
        }
        W.bnd[lvl - 1][lane] = b;
        if (lane == 0) {
            W.mask[lvl] = mt;
            W.base[lvl] = first;
        }
        wave_lds_sync();
    }
}

// Reductions over the 32 lanes of each half, every lane receiving its half's:
// rotations within rows of 16 lanes, then the half's two rows.
template <class T, class Op>
__device__ __forceinline__ T half_reduce(T v, Op op)
{
    auto ror = [](T x, auto ctl) {
        return __builtin_bit_cast(T, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(uint32_t, x), decltype(ctl)::value, 0xF,
                                                              0xF, true));
    };
    v = op(v, ror(v, std::integral_constant<int, 0x128>()));   // row_ror:8
    v = op(v, ror(v, std::integral_constant<int, 0x124>()));
    v = op(v, ror(v, std::integral_constant<int, 0x122>()));
    v = op(v, ror(v, std::integral_constant<int, 0x121>()));
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const uint32_t a = r[0], b = r[1];
    return op(__builtin_bit_cast(T, a), __builtin_bit_cast(T, b));
}
__device__ __forceinline__ float half_max(float v)
{
    return half_reduce(v, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float half_min(float v)
{
    return half_reduce(v, [](float a, float b) { return fminf(a, b); });
}
__device__ __forceinline__ uint32_t half_sum(uint32_t v)
{
    return half_reduce(v, [](uint32_t a, uint32_t b) { return a + b; });
}

// Query q's list of cnt keys (unsorted) and a tile's further cnew <= 32 keys:
// the CAP smallest of both, sorted, into the list; returns the kp-th score.
// Whole wavefront.
template <int E>
__device__ __noinline__ float overflow_list(uint64_t* __restrict__ dst, int cnt, const uint64_t* buf, int cnew, int kp)
{
    const int lane = lane_id();
    uint64_t L[E];
#pragma unroll
    for (int s = 0; s < E; ++s) L[s] = s * WAVE + lane < cnt ? dst[s * WAVE + lane] : KEY_INF;
    uint64_t B[1] = {lane >= 32 && lane - 32 < cnew ? buf[lane - 32] : KEY_INF};
    bitonic_sort<E>(L);
    // the new keys descending in the upper half: reversed ascending order
#pragma unroll
    for (int kb = 2; kb <= 32; kb <<= 1) {
#pragma unroll
        for (int j = kb >> 1; j > 0; j >>= 1) cx_lanes<1>(B, kb, j, lane);
    }
    L[E - 1] = umin64(L[E - 1], B[0]);
    bitonic_merge_asc<E>(L);
#pragma unroll
    for (int s = 0; s < E; ++s) dst[s * WAVE + lane] = L[s];
    return key_dist(list_at<E>(L, kp - 1));
}

// A list of cnt keys (unsorted, CAP - 32 < cnt) cut: the keys above tau are dropped,
// and while more than kp + (CAP - kp) / 4 are left, those above a lower threshold that at
// least kp do not exceed. Returns the count in the upper half and the threshold's
// bits; nothing is dropped where equal scores leave no such threshold. Whole wavefront.
template <int E>
__device__ __noinline__ uint64_t cut_list(uint64_t* __restrict__ dst, int cnt, int kp, float tau)
{
    const int lane = lane_id();
    const int most = kp + (WAVE * E - kp) / 4;
    uint64_t v[E];
    uint32_t d[E];
    uint32_t first = ~0u;
#pragma unroll
    for (int s = 0; s < E; ++s) {
        v[s] = s * WAVE + lane < cnt ? dst[s * WAVE + lane] : ~0ull;
        d[s] = static_cast<uint32_t>(v[s] >> 32);
        first = min(first, d[s]);
    }
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) first = min(first, static_cast<uint32_t>(xor_lane(first, o)));
    auto count = [&](uint32_t t) {
        int c = 0;
#pragma unroll
        for (int s = 0; s < E; ++s) c += __popcll(__ballot(d[s] <= t));
        return c;
    };
    // as ordered bits; lo: fewer than kp scores do not exceed it; hi: at many do not
    uint32_t lo = __builtin_amdgcn_readfirstlane(first) - 1u;
    uint32_t hi = __builtin_amdgcn_readfirstlane(float_order_bits(tau));
    int at = count(hi);
    while (at > most && hi - lo > 1u) {
        // the middle of the values, or of the bits where rounding leaves it at an end
        const float a = order_bits_float(lo), b = order_bits_float(hi);
        uint32_t mid = __builtin_amdgcn_readfirstlane(float_order_bits(a + 0.5f * (b - a)));
        if (!(mid > lo && mid < hi)) mid = lo + (hi - lo) / 2;
        const int c = count(mid);
        if (c < kp) {
            lo = mid;
        } else {
            hi = mid;
            at = c;
        }
    }
    if (at > most) return static_cast<uint64_t>(cnt) << 32 | __float_as_uint(tau);
    int w = 0;
#pragma unroll
    for (int s = 0; s < E; ++s) {
        const uint64_t mask = __ballot(d[s] <= hi);
        if (d[s] <= hi) dst[w + mbcnt64(mask)] = v[s];
        w += __popcll(mask);
    }
    return static_cast<uint64_t>(w) << 32 | __float_as_uint(order_bits_float(hi));
}

// A list of cnt keys sorted, the places behind them filled; returns the kp-th
// score. Whole wavefront.
template <int E>
__device__ __noinline__ float sort_list(uint64_t* __restrict__ dst, int cnt, int kp)
{
    const int lane = lane_id();
    uint64_t L[E];
#pragma unroll
    for (int s = 0; s < E; ++s) L[s] = s * WAVE + lane < cnt ? dst[s * WAVE + lane] : KEY_INF;
    bitonic_sort<E>(L);
#pragma unroll
    for (int s = 0; s < E; ++s) dst[s * WAVE + lane] = L[s];
    return key_dist(list_at<E>(L, kp - 1));
}

// Bound on the error of the scores of a query of squared norm yi2 (E_i), and the
// lower bound on the squared distance of its candidates with a score at or above s.
__device__ __forceinline__ double score_error(float yi2, float R, const ErrModel& em)
{
    const double Rd = static_cast<double>(R), yi = sqrt(static_cast<double>(yi2));
    return em.gamma * (Rd + 1.05 * yi) * (Rd + 1.05 * yi) + em.norm * Rd * Rd + em.cross * yi * Rd + 1e-30;
}
__device__ __forceinline__ float certificate_bound(float s, float yi2, float R, const ErrModel& em)
{
    const double t = static_cast<double>(s) + static_cast<double>(yi2) - score_error(yi2, R, em);
    double B = t > 0.0 ? sqrt(t) : 0.0;
    B -= em.center * (sqrt(static_cast<double>(yi2)) + static_cast<double>(R));
    B = B > 0.0 ? B : 0.0;
    return static_cast<float>(B * B * (1.0 - 1.0 / 1048576.0));
}

// stores of this wavefront complete before its later loads read them
__device__ __forceinline__ void wave_global_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

}  // namespace

// K-steps of a long product's batch of loads: all of up to 15 BF16 (32 FP32)
// fragments, else BF16 in halves and FP32 in equal batches of at most 32.
template <class Tr, int KS>
constexpr int tree_batch()
{
    constexpr int most = sizeof(typename Tr::frag) == 16 ? 16 : 32;
    constexpr int nb = (KS + most - 1) / most;
    return sizeof(typename Tr::frag) == 16 && KS >= 16 ? (KS + 1) / 2 : (KS + nb - 1) / nb;
}

// The lists' room: CAP = 64 E keys. BUF: kp may be within 32 of it, a full list is
// kept sorted and takes further keys from a buffer; else it is cut.
template <class Tr, int KS, bool LONG>
constexpr size_t tree_operand_bytes()
{
    return LONG ? static_cast<size_t>(KS) * WAVE * sizeof(typename Tr::frag) : 0;
}

template <class Tr, int KS, bool LONG, int E, int D, bool BUF, int WPE>
__global__ __launch_bounds__(WAVE, WPE) void k_select_tree(
    const typename Tr::elem* __restrict__ Aq, const typename Tr::elem* __restrict__ Bc, int n, int kp,
    const float* __restrict__ ynorm2, const unsigned* __restrict__ rmax_bits, ErrModel em,
    uint64_t* __restrict__ lists, float* __restrict__ lb_out, CurveArgs crv, int probe, int wide_min,
    unsigned long long* __restrict__ pair_count)
{
    using elem = typename Tr::elem;
    using frag = typename Tr::frag;
    constexpr int kpad = KS * Tr::KSTEP;
    constexpr int KR = LONG ? 1 : KS;           // fragments of a tile kept in registers
    constexpr int CAP = WAVE * E;
    constexpr int FILL = CAP / 32;
    // the notes; fewer where the operand and the buffers would leave room for only three wavefronts per CU
    constexpr int NOTES = LONG && BUF ? 224 : 384;
    __shared__ TreeLds<NOTES> W;
    __shared__ TreeShape s_shape;
    extern __shared__ __attribute__((aligned(16))) char s_dyn[];
    frag* s_a = reinterpret_cast<frag*>(s_dyn);   // LONG: the query operand, [k-step][lane]
    // BUF: each query's buffer of TBUF keys and its count (-1: the list is not
    // sorted yet); else a tile's keys that a list has no room for, per half
    uint64_t* s_keys = reinterpret_cast<uint64_t*>(s_dyn + tree_operand_bytes<Tr, KS, LONG>());
    int* s_nbuf = reinterpret_cast<int*>(s_keys + TNQ * TBUF);

    const int lane = lane_id();
    const int half = lane >> 5, l31 = lane & 31;
    if (threadIdx.x == 0) {
        s_shape.top = crv.layout.top;
        for (int l = 0; l < TREE_LEVELS; ++l) {
            s_shape.cnt[l] = crv.layout.cnt[l];
            s_shape.off[l] = crv.layout.off[l];
        }
    }
    const int ntiles = crv.layout.cnt[0];
    // this wavefront's query tile
    const int t0 = probe ? static_cast<int>(static_cast<int64_t>(blockIdx.x) * ntiles / gridDim.x) : xcd_block();
    const int q0 = t0 * TNQ;
    const int nq_valid = min(TNQ, n - q0);
    uint64_t* lists_q0 = lists + static_cast<size_t>(q0) * CAP;

    // query fragments: curve position q0 + l31 (the last tile's padding rows
    // repeat a real row; their results are never stored)
    frag qa[KR];
    {
        const elem* src = Aq + static_cast<size_t>(min(q0 + l31, n - 1)) * kpad + half * Tr::VEC;
        if constexpr (LONG) {
#pragma unroll 8
            for (int s = 0; s < KS; ++s) s_a[s * WAVE + lane] = Tr::load(src + s * Tr::KSTEP);
        } else {
#pragma unroll
            for (int s = 0; s < KS; ++s) qa[s] = Tr::load(src + s * Tr::KSTEP);
        }
    }
    const float R = __uint_as_float(*rmax_bits);
    BoxBound bb;
    bb.zerr = crv.zcoef * R;
    bb.pscale = *crv.pscale;
    bb.yerr = crv.ycoef * R;
    // LONG: the queries' projected operand for the pairwise bound, split into
    // BF16 terms: [-2 hi | -2 hi], [-2 lo | 1 1 1 0...] (lane halves), against the
    // candidates' [hi | lo], [hi | |z|^2 in three terms]; and the part of a
    // query's projected threshold that does not change.
    bf16x8 za0 = {}, za1 = {};
    float zconst = 0.f;   // lane q < 32: E_q - |z_q|^2
    const float zslack = 2.f * 2.8285f * bb.zerr;   // sqrt(PR_DIMS) zerr at either end of a projected distance
    PointTest pt;
    {
        const float4* src = reinterpret_cast<const float4*>(crv.zs + static_cast<size_t>(min(q0 + l31, n - 1)) * PR_DIMS);
        const float4 u = src[0], v = src[1];
        pt.z[0] = half ? v.x : u.x;
        pt.z[1] = half ? v.y : u.y;
        pt.z[2] = half ? v.z : u.z;
        pt.z[3] = half ? v.w : u.w;
        pt.gt = TINF;
        if constexpr (LONG) {
            const float z[PR_DIMS] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
            float z2 = 0.f;
#pragma unroll
            for (int c = 0; c < PR_DIMS; ++c) {
                const __bf16 hi = static_cast<__bf16>(z[c]);
                const __bf16 lo = static_cast<__bf16>(z[c] - static_cast<float>(hi));
                z2 = fmaf(z[c], z[c], z2);
                za0[c] = static_cast<__bf16>(-2.f * static_cast<float>(hi));
                za1[c] = half ? static_cast<__bf16>(c < 3 ? 1.f : 0.f)
                              : static_cast<__bf16>(-2.f * static_cast<float>(lo));
            }
            // Error of the computed s' = |z_j|^2 - 2 z_i.z_j: the terms left
            // out of the BF16 split are below 3.1 2^-18 |z_i| |z_j| (twice that
            // in s'), the accumulation below 36 2^-24 (|z_j|^2 + 2.1 |z_i| |z_j|),
            // the norm's rounding 10 2^-24 |z_j|^2, and |z_q|^2 here errs by
            // 8 2^-24 |z_q|^2.
            const float rz = (R / bb.pscale + 3.f * bb.zerr) * (1.f + 1e-5f);
            zconst = 3.5e-5f * sqrtf(z2) * rz + 4e-6f * rz * rz - z2;
        }
    }
    if (lane < 2 * PR_DIMS) W.box[lane] = crv.tbox[static_cast<size_t>(t0) * 2 * PR_DIMS + lane];
    if (lane < TNQ) {
        W.yq[lane] = lane < nq_valid ? ynorm2[q0 + lane] : 0.f;
        W.tau[lane] = lane < nq_valid ? TINF : -TINF;
        if constexpr (BUF) s_nbuf[lane] = -1;
    }
    __syncthreads();

    // the distance threshold of a score threshold (rounded up)
    auto dist_threshold = [](float score, float yq) { return fmaxf(score + yq, 0.f) * (1.f + 4.8e-7f); };
    // distance thresholds and, LONG, projected thresholds from W.tau (`counted`:
    // those of every candidate whose computed score is at or below it); returns
    // the wavefront's largest distance threshold (read from one lane, so that
    // the compiler sees a wave-uniform value and keeps the branches on it,
    // and the state they update, scalar).
    // |x_i - x_j|^2 <= thr implies |z_i - z_j| <= (sqrt(thr) + yerr) / pscale + zslack
    // (see BoxBound), hence s' <= that^2 - |z_i|^2 + E_i.
    auto publish = [&](bool counted) {
        wave_lds_sync();
        float t = -TINF;
        if (lane < TNQ) {
            t = lane < nq_valid ? dist_threshold(W.tau[lane], W.yq[lane]) : -TINF;
            auto projected = [&](float d2) {
                const float b = (sqrtf(fmaxf(d2, 0.f)) * (1.f + 1e-6f) + bb.yerr) / bb.pscale + zslack;
                return b * b * (1.f + 4e-6f);
            };
            W.gt[lane] = lane < nq_valid ? projected(t) : -TINF;
            if constexpr (LONG) {
                const float tz = counted ? t + static_cast<float>(score_error(W.yq[lane], R, em) * (1.0 + 1e-6)) : t;
                W.zt[lane] = lane < nq_valid ? projected(tz) + zconst : -TINF;
            }
        }
        wave_lds_sync();
        pt.gt = W.gt[l31];
        return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(wave_max_f32(t))));
    };
    // this lane's 16 rows of a per-query LDS array (four consecutive per group)
    auto rows16 = [&](const float* a, float (&v)[16]) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 t = *reinterpret_cast<const float4*>(a + 8 * g + 4 * half);
            v[4 * g] = t.x;
            v[4 * g + 1] = t.y;
            v[4 * g + 2] = t.z;
            v[4 * g + 3] = t.w;
        }
    };

    auto load_tile = [&](int t, frag (&b)[KR]) {
        const elem* src = Bc + static_cast<size_t>(t) * 32 * kpad + lane * Tr::VEC;
#pragma unroll
        for (int s = 0; s < KR; ++s) b[s] = Tr::load(src + s * 64 * Tr::VEC);
    };
    // one accumulator chain
    auto product = [&](const frag (&b)[KR]) {
        f32x16 a = {};
#pragma unroll
        for (int s = 0; s < KR; ++s) a = Tr::mma(qa[s], b[s], a);
        return a;
    };
    // the long product: the tile's fragments in batches of U K-steps, with one
    // wavefront per SIMD the next batch's loads in flight during a batch's
    // products; even and odd K-steps in two accumulators
    auto product_long = [&](int t) {
        constexpr int U = tree_batch<Tr, KS>(), NB = (KS + U - 1) / U;
        constexpr int AHEAD = WPE == 1 && NB > 1 ? 2 : 1;
        const elem* src = Bc + static_cast<size_t>(t) * 32 * kpad + lane * Tr::VEC;
        f32x16 acc0 = {}, acc1 = {};
        frag b[AHEAD][U];
#pragma unroll
        for (int u = 0; u < U; ++u) b[0][u] = Tr::load(src + u * 64 * Tr::VEC);
#pragma unroll
        for (int g = 0; g < NB; ++g) {
            if (AHEAD == 1 && g > 0) {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (g * U + u < KS) b[0][u] = Tr::load(src + (g * U + u) * 64 * Tr::VEC);
            }
            if (AHEAD == 2) {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if ((g + 1) * U + u < KS) b[(g + 1) % AHEAD][u] = Tr::load(src + ((g + 1) * U + u) * 64 * Tr::VEC);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = g * U + u;
                if (k >= KS) continue;
                if (k % 2 == 0)
                    acc0 = Tr::mma(s_a[k * WAVE + lane], b[g % AHEAD][u], acc0);
                else
                    acc1 = Tr::mma(s_a[k * WAVE + lane], b[g % AHEAD][u], acc1);
            }
        }
        return KS > 1 ? acc0 + acc1 : acc0;
    };
    auto scores = [&](int t, const frag (&b)[KR]) {
        if constexpr (LONG)
            return product_long(t);
        else
            return product(b);
    };

    // ================================================================ pass 1
    // top[r][0..D-1]: the D smallest scores seen by this lane for its query acc_row(r, half), ascending
    float top[16][D];
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int d = 0; d < D; ++d) top[r][d] = TINF;
    const int qd = (kp + 31) / 32 - 1;   // every lane's (qd + 1)-th smallest: at least kp scores up to the largest of them
    // new thresholds from top; tau never rises
    auto refresh = [&](int iters) {
        float old[16];
        rows16(W.tau, old);
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            float lo[2], hi[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                float v = top[r + u][0];
#pragma unroll
                for (int d = 1; d < D; ++d)
                    if (d == qd) v = top[r + u][d];
                hi[u] = half_max(v);
                lo[u] = half_min(v);
                if (__ballot(hi[u] == TINF)) {
                    // a lane with fewer scores: search up to the largest score there is
                    float m = -TINF;
#pragma unroll
                    for (int d = 0; d < D; ++d) m = top[r + u][d] < TINF ? fmaxf(m, top[r + u][d]) : m;
                    m = half_max(m);
                    const float f = half_min(top[r + u][0]);
                    lo[u] = hi[u] == TINF ? f : lo[u];
                    hi[u] = hi[u] == TINF ? m : hi[u];
                }
                hi[u] = fminf(hi[u], old[r + u]);
            }
            auto counts = [&](float a, float b) {
                uint32_t c = 0;
#pragma unroll
                for (int d = 0; d < D; ++d) c += (top[r][d] <= a ? 1u : 0u) + (top[r + 1][d] <= b ? 65536u : 0u);
                return half_sum(c);
            };
            for (int it = 0; it < iters; ++it) {
                const float m0 = lo[0] + 0.5f * (hi[0] - lo[0]), m1 = lo[1] + 0.5f * (hi[1] - lo[1]);
                const uint32_t c = counts(m0, m1);
                const bool g0 = static_cast<int>(c & 0xFFFFu) >= kp, g1 = static_cast<int>(c >> 16) >= kp;
                hi[0] = g0 ? m0 : hi[0];
                lo[0] = g0 ? lo[0] : m0;
                hi[1] = g1 ? m1 : hi[1];
                lo[1] = g1 ? lo[1] : m1;
            }
            // a threshold needs kp scores at or below it (fewer seen so far: none yet)
            const uint32_t c = counts(hi[0], hi[1]);
            const float t0n = static_cast<int>(c & 0xFFFFu) >= kp ? hi[0] : old[r];
            const float t1n = static_cast<int>(c >> 16) >= kp ? hi[1] : old[r + 1];
            if (l31 == 0) {
                W.tau[acc_row(r, half)] = t0n;
                W.tau[acc_row(r + 1, half)] = t1n;
            }
        }
        return publish(false);
    };
    unsigned long long pairs = 0;
    int nrec = 0;       // tiles noted (at most NOTES)
    int pend = 0;       // noted since the last refresh
    auto take_scores = [&](const f32x16& acc, int tile) {
        const int cand = tile * 32 + l31;
        const bool valid = cand < n;
        pairs += static_cast<unsigned long long>(nq_valid) * __popcll(__ballot(valid) & 0xFFFFFFFFull);
        float tv[16];
        rows16(W.tau, tv);
        bool hit = false;
#pragma unroll
        for (int r = 0; r < 16; ++r) hit |= acc[r] <= tv[r];
        if (!__ballot(valid && hit)) return;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            // sorted insertion: top[d] = median(top[d - 1], x, top[d])
            const float x = valid && acc[r] <= tv[r] ? acc[r] : TINF;
#pragma unroll
            for (int d = D - 1; d > 0; --d) top[r][d] = __builtin_amdgcn_fmed3f(top[r][d - 1], x, top[r][d]);
            top[r][0] = fminf(top[r][0], x);
        }
        if (lane == 0) W.rec[nrec] = static_cast<uint32_t>(tile);
        ++nrec;
        ++pend;
    };

    // the FILL tiles around the own tile
    const int nfill = min(FILL, ntiles);
    const int f0 = max(0, min(t0 - (FILL / 2 - 1), ntiles - nfill));
    for (int i = 0; i < nfill; ++i) {
        frag b[KR];
        if constexpr (!LONG) load_tile(f0 + i, b);
        take_scores(scores(f0 + i, b), f0 + i);
    }
    // every fill tile is noted (its candidates may all lie beyond infinite scores only if none is valid)
    float wthr = refresh(6);
    pend = 0;

    // ---- tree walk: the current group of tiles in registers, the levels above in LDS
    TileGroup g = {0ull, 0, __builtin_nanf("")};
    auto walk_start = [&]() {
        bool take;
        if (s_shape.top == 0) {
            g.base = 0;
            g.bnd = child_bound(crv.tbox, crv.tree, &s_shape, 0, 0, W.box, bb, f0, nfill, W.gbox, take);
            g.mask = __ballot(take);
            if (lane == 0) W.lvl = 0;
        } else {
            const int top_l = s_shape.top;
            g.mask = 0ull;
            W.bnd[top_l - 1][lane] = child_bound(crv.tbox, crv.tree, &s_shape, top_l, 0, W.box, bb, f0, nfill,
                                                W.gbox, take);
            const uint64_t mt = __ballot(take);
            if (lane == 0) {
                W.mask[top_l] = mt;
                W.base[top_l] = 0;
                W.lvl = top_l;
            }
        }
        wave_lds_sync();
    };
    // next tile within reach of thr (and its bound), or -1
    auto next_tile = [&](float thr, float& tb) -> int {
        while (true) {
            const uint64_t m = g.mask & __ballot(g.bnd <= thr);
            if (m) {
                const int c = nearest_lane(m, g.bnd);
                g.mask = m & ~(1ull << c);
                const float4* gb = reinterpret_cast<const float4*>(W.gbox[c]);
                if (!pt.reach(gb[half], gb[PR_DIMS / 4 + half])) continue;
                tb = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(g.bnd), c));
                return g.base + c;
            }
            g = climb(W, &s_shape, crv.tbox, crv.tree, bb, pt, thr, f0, nfill);
            if (g.base < 0) return -1;
        }
    };
    // LONG: whether some pair of the tile is within reach by its projections
    auto load_z = [&](int t, float4 (&z)[2]) {
        const float4* src = reinterpret_cast<const float4*>(crv.zs + (static_cast<size_t>(t) * 32 + l31) * PR_DIMS);
        z[0] = src[0];
        z[1] = src[1];
    };
    auto z_reach = [&](const float4 (&zz)[2], int tile) -> bool {
        const float z[PR_DIMS] = {zz[0].x, zz[0].y, zz[0].z, zz[0].w, zz[1].x, zz[1].y, zz[1].z, zz[1].w};
        bf16x8 hi, lo, nz;
        float z2 = 0.f;
#pragma unroll
        for (int c = 0; c < PR_DIMS; ++c) {
            hi[c] = static_cast<__bf16>(z[c]);
            lo[c] = static_cast<__bf16>(z[c] - static_cast<float>(hi[c]));
            z2 = fmaf(z[c], z[c], z2);
            nz[c] = static_cast<__bf16>(0.f);
        }
        nz[0] = static_cast<__bf16>(z2);
        const float r1 = z2 - static_cast<float>(nz[0]);
        nz[1] = static_cast<__bf16>(r1);
        nz[2] = static_cast<__bf16>(r1 - static_cast<float>(nz[1]));
        const bf16x8 b0 = half ? lo : hi, b1 = half ? nz : hi;
        f32x16 a = {};
        a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(za0, b0, a, 0, 0, 0);
        a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(za1, b1, a, 0, 0, 0);
        float tv[16];
        rows16(W.zt, tv);
        bool hit = false;
#pragma unroll
        for (int r = 0; r < 16; ++r) hit |= a[r] <= tv[r];
        return __ballot(tile * 32 + l31 < n && hit) != 0ull;
    };

    // how many of 64 tiles spread over the samples are within reach of some query
    auto sampled_reach = [&]() {
        const int v = static_cast<int>(static_cast<int64_t>(lane) * ntiles / WAVE);
        float b[2 * PR_DIMS];
        load_box(crv.tbox + static_cast<size_t>(v) * 2 * PR_DIMS, b);
        bool in = false;
        for (int q = 0; q < nq_valid; ++q) {
            float g2 = 0.f;
#pragma unroll
            for (int c = 0; c < PR_DIMS; ++c) {
                const float z = __int_as_float(
                    __builtin_amdgcn_readlane(__float_as_int(pt.z[c % 4]), q + 32 * (c / 4)));
                const float g = fmaxf(fmaxf(b[c] - z, z - b[PR_DIMS + c]), 0.f);
                g2 = fmaf(g, g, g2);
            }
            in = in || g2 <= W.gt[q];
        }
        return __popcll(__ballot(in));
    };
    constexpr int DEPTH = TREE_DEPTH;
    constexpr int ZR = LONG ? DEPTH : 1, BR = LONG ? 1 : DEPTH;
    int tq[DEPTH];         // the tiles in flight, the current one first (-1: none)
    float tbq[DEPTH];      // their bounds when taken
    frag bq[BR][KR];       // their fragments
    float4 zq[ZR][2];      // LONG: their projections
    auto fetch = [&](int d) {
        if (tq[d] < 0) return;
        if constexpr (LONG)
            load_z(tq[d], zq[d]);
        else
            load_tile(tq[d], bq[d]);
    };
    auto shift = [&]() {
#pragma unroll
        for (int d = 0; d + 1 < DEPTH; ++d) {
            tq[d] = tq[d + 1];
            tbq[d] = tbq[d + 1];
            if constexpr (LONG) {
                zq[d][0] = zq[d + 1][0];
                zq[d][1] = zq[d + 1][1];
            } else {
#pragma unroll
                for (int s = 0; s < KR; ++s) bq[d][s] = bq[d + 1][s];
            }
        }
    };
    auto pipe_start = [&](auto next) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            tq[d] = -1;
            tbq[d] = 0.f;
        }
#pragma unroll
        for (int s = 0; s < BR; ++s)
#pragma unroll
            for (int t = 0; t < KR; ++t) bq[s][t] = {};
#pragma unroll
        for (int d = 0; d < ZR; ++d) zq[d][0] = zq[d][1] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int d = 0; d + 1 < DEPTH; ++d) {
            if (d == 0 || tq[d - 1] >= 0) tq[d] = next(tbq[d]);
            fetch(d);
        }
    };
    auto walk_next = [&](float& tb) { return next_tile(wthr, tb); };
    walk_start();
    pipe_start(walk_next);
    // a launch of 64 query tiles spread over the samples adds up their reach by the
    // thresholds of the fill (looser than a walk's)
    if (probe) {
        const int reach = sampled_reach();
        if (lane == 0) atomicAdd(crv.wide_count + 1, reach);
        return;
    }
    const bool wide = crv.wide_count[1] > wide_min;
    const int notes = wide ? TASK : NOTES;
    while (tq[0] >= 0 && nrec < notes) {
        tq[DEPTH - 1] = tq[DEPTH - 2] >= 0 ? walk_next(tbq[DEPTH - 1]) : -1;
        fetch(DEPTH - 1);
        // the current tile may have fallen out of reach since it was taken
        bool reach = tbq[0] <= wthr;
        if constexpr (LONG) reach = reach && z_reach(zq[0], tq[0]);
        if (reach) {
            take_scores(scores(tq[0], bq[0]), tq[0]);
            if (pend >= 4 + (nrec >> 2)) {
                wthr = refresh(6);
                pend = 0;
            }
        }
        shift();
    }
    wthr = refresh(9);
    if (wide && tq[0] >= 0) {   // the scans start from these thresholds
        if (lane < nq_valid) lb_out[q0 + lane] = W.tau[lane];
        if (lane == 0) crv.wide[atomicAdd(crv.wide_count, 1)] = t0;
        return;
    }

    // ================================================================ pass 2
    int at[16];   // the next free key of this half's queries' lists (from lists_q0)
#pragma unroll
    for (int r = 0; r < 16; ++r) at[r] = acc_row(r, half) * CAP;
    // the noted tiles and those in flight when the notes were full, then the rest of the walk
    const bool more = tq[0] >= 0;
    int nlist = nrec;
#pragma unroll
    for (int d = 0; d + 1 < DEPTH; ++d) {
        if (tq[d] < 0) continue;
        if (lane == 0) W.rec[nlist] = static_cast<uint32_t>(tq[d]);
        ++nlist;
    }
    if constexpr (LONG)
        publish(true);
    else
        wave_lds_sync();
    int ri = 0;
    auto list_next = [&](float& tb) -> int {
        tb = 0.f;
        if (ri < nlist) return __builtin_amdgcn_readfirstlane(static_cast<int>(W.rec[ri++]));
        return more ? next_tile(wthr, tb) : -1;
    };
    int fell = 0;   // thresholds lowered since they were last published
    pipe_start(list_next);
    for (int done = 0; tq[0] >= 0; ++done) {
        if (done >= nlist && (done == nlist || fell >= 8)) {   // beyond the noted tiles
            wthr = publish(false);
            fell = 0;
        }
        tq[DEPTH - 1] = tq[DEPTH - 2] >= 0 ? list_next(tbq[DEPTH - 1]) : -1;
        fetch(DEPTH - 1);
        bool reach = tbq[0] <= wthr;
        if constexpr (LONG) reach = reach && z_reach(zq[0], tq[0]);
        if (reach) {
            const int cand = tq[0] * 32 + l31;
            const bool valid = cand < n;
            if (done >= nrec)
                pairs += static_cast<unsigned long long>(nq_valid) * __popcll(__ballot(valid) & 0xFFFFFFFFull);
            const f32x16 acc = scores(tq[0], bq[0]);
            float tv[16];
            rows16(W.tau, tv);
            const uint32_t below = (1u << l31) - 1u;
            uint32_t missed = 0;   // rows whose list has no room: not stored here
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const bool in = valid && acc[r] <= tv[r];
                const uint64_t mask = __ballot(in);
                if (!mask) continue;
                const uint32_t mh = half ? static_cast<uint32_t>(mask >> 32) : static_cast<uint32_t>(mask);
                const int next = at[r] + __popc(mh), slot = at[r] + __popc(mh & below);
                const bool room = next <= (acc_row(r, half) + 1) * CAP;
                missed |= room ? 0u : 1u << r;
                if (in && room) lists_q0[slot] = make_key(acc[r], static_cast<uint32_t>(cand));
                at[r] = room ? next : at[r];
            }
            if (__ballot(missed != 0)) {
                wave_lds_sync();
                wave_global_sync();
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const bool over = (missed >> r) & 1u;
                    const uint64_t om = __ballot(over);   // by half
                    if (!om) continue;
                    const int qh = acc_row(r, half);
                    auto keys_of = [&](float t, uint32_t& mh) {   // this tile's keys of the full lists
                        const bool in = over && valid && acc[r] <= t;
                        const uint64_t mask = __ballot(in);
                        mh = half ? static_cast<uint32_t>(mask >> 32) : static_cast<uint32_t>(mask);
                        return in;
                    };
                    uint32_t mh;
                    bool in = keys_of(tv[r], mh);
                    if constexpr (BUF) {
                        const int b = s_nbuf[qh];
                        const uint64_t make = __ballot(over && (b < 0 || b + __popc(mh) > TBUF));
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            if (!((make >> (32 * h)) & 1ull)) continue;
                            const int q = acc_row(r, h);
                            uint64_t* dst = lists_q0 + static_cast<size_t>(q) * CAP;
                            const int bq = __builtin_amdgcn_readlane(b, 32 * h);
                            const float nt =
                                bq < 0 ? sort_list<E>(dst, __builtin_amdgcn_readlane(at[r], 32 * h) - q * CAP, kp)
                                       : merge_query_list<E>(dst, s_keys + q * TBUF, bq, kp);
                            wave_lds_sync();
                            if (lane == 0) {
                                W.tau[q] = fminf(W.tau[q], nt);
                                s_nbuf[q] = 0;
                            }
                            if (half == h) at[r] = (q + 1) * CAP;
                            ++fell;
                        }
                        wave_lds_sync();
                        in = keys_of(W.tau[qh], mh);
                        const int nb = s_nbuf[qh];
                        if (in) s_keys[qh * TBUF + nb + __popc(mh & below)] = make_key(acc[r], static_cast<uint32_t>(cand));
                        wave_lds_sync();
                        if (over && l31 == 0) s_nbuf[qh] = nb + __popc(mh);
                        wave_lds_sync();
                    } else {
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            if (!((om >> (32 * h)) & 1ull)) continue;
                            const int q = acc_row(r, h);
                            const uint64_t cut = cut_list<E>(lists_q0 + static_cast<size_t>(q) * CAP,
                                                             __builtin_amdgcn_readlane(at[r], 32 * h) - q * CAP, kp,
                                                             W.tau[q]);
                            if (lane == 0) W.tau[q] = __uint_as_float(static_cast<uint32_t>(cut));
                            if (half == h) at[r] = q * CAP + static_cast<int>(cut >> 32);
                            ++fell;
                        }
                        wave_lds_sync();
                        in = keys_of(W.tau[qh], mh);
                        const int next = at[r] + __popc(mh), slot = at[r] + __popc(mh & below);
                        const bool room = next <= (qh + 1) * CAP;
                        if (in && room) lists_q0[slot] = make_key(acc[r], static_cast<uint32_t>(cand));
                        const uint64_t full = __ballot(over && !room);
                        if (over && room) at[r] = next;
                        if (full) {   // equal scores fill the list
                            if (in) s_keys[half * TNQ + __popc(mh & below)] = make_key(acc[r], static_cast<uint32_t>(cand));
                            wave_lds_sync();
                            wave_global_sync();
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                if (!((full >> (32 * h)) & 1ull)) continue;
                                const int q = acc_row(r, h);
                                const int c = __builtin_amdgcn_readlane(at[r], 32 * h) - q * CAP;
                                const int add = __popc(__builtin_amdgcn_readlane(mh, 32 * h));
                                const float nt = overflow_list<E>(lists_q0 + static_cast<size_t>(q) * CAP, c,
                                                                  s_keys + h * TNQ, add, kp);
                                if (lane == 0) W.tau[q] = fminf(W.tau[q], nt);
                                if (half == h) at[r] = (q + 1) * CAP;
                            }
                            wave_lds_sync();
                        }
                    }
                }
                wave_global_sync();
            }
        }
        shift();
    }
    // the lists' stores complete before other lanes read them
    wave_lds_sync();
    wave_global_sync();
    if constexpr (BUF) {
        for (int q = 0; q < nq_valid; ++q) {
            const int b = __builtin_amdgcn_readfirstlane(s_nbuf[q]);
            if (b > 0) merge_query_list<E>(lists_q0 + static_cast<size_t>(q) * CAP, s_keys + q * TBUF, b, kp);
        }
        wave_global_sync();
    }
    // each list sorted in place, the next one's loads in flight meanwhile;
    // query q's count moved to lane q
    int cnt_lane = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int c0 = __builtin_amdgcn_readlane(at[r], 0), c1 = __builtin_amdgcn_readlane(at[r], 32);
        if (lane == acc_row(r, 0)) cnt_lane = c0 - lane * CAP;
        if (lane == acc_row(r, 1)) cnt_lane = c1 - lane * CAP;
    }
    {
        auto load_list = [&](int q, uint64_t (&L)[E]) {
            const int c = __builtin_amdgcn_readlane(cnt_lane, q);
#pragma unroll
            for (int s = 0; s < E; ++s)
                L[s] = s * WAVE + lane < c ? lists_q0[static_cast<size_t>(q) * CAP + s * WAVE + lane] : KEY_INF;
        };
        uint64_t Ln[E];
        load_list(0, Ln);
        for (int q = 0; q < nq_valid; ++q) {
            uint64_t L[E];
#pragma unroll
            for (int s = 0; s < E; ++s) L[s] = Ln[s];
            if (q + 1 < nq_valid) load_list(q + 1, Ln);
            bitonic_sort<E>(L);
#pragma unroll
            for (int s = 0; s < E; ++s) lists_q0[static_cast<size_t>(q) * CAP + s * WAVE + lane] = L[s];
            // the list's kp-th score (+inf where it is short), for the certificate below
            const float sl = key_dist(list_at<E>(L, kp - 1));
            if (lane == 0) W.tau[q] = fminf(sl, W.tau[q]);
        }
        wave_lds_sync();
    }
    count_pairs(pair_count, pairs);

    // certificate lower bound for the candidates left out of each list
    if (lane < nq_valid) lb_out[q0 + lane] = certificate_bound(W.tau[lane], W.yq[lane], R, em);
}

// The query tiles of short contractions that k_select_tree handed over (crv.wide),
// a wavefront each: many tiles are within reach, so there is little to walk or to
// note. Every tile within reach by its box (and, unless all sampled ones were, by the
// single queries) is scored once, 64 boxes bounded at a time from the own group on;
// lists start empty from the thresholds in lb_out and take keys from buffers in
// LDS, TBUF at a time. Bound by the latency of a tile's chain (box tests, products,
// compares); without kept scores the registers hold up to four wavefronts per
// SIMD instead of two, which is what this form is for (tree_wide_min).
template <class Tr, int KS>
constexpr int scan_waves()
{
    constexpr int fr = TREE_DEPTH * KS * static_cast<int>(sizeof(typename Tr::frag) / 4);
    return fr <= 36 ? 4 : fr <= 64 ? 3 : 2;
}

template <class Tr, int KS, int E>
__global__ __launch_bounds__(WAVE, (scan_waves<Tr, KS>())) void k_select_scan(
    const typename Tr::elem* __restrict__ Aq, const typename Tr::elem* __restrict__ Bc, int n, int kp,
    const float* __restrict__ ynorm2, const unsigned* __restrict__ rmax_bits, ErrModel em,
    uint64_t* __restrict__ lists, float* __restrict__ lb_out, CurveArgs crv,
    unsigned long long* __restrict__ pair_count)
{
    using elem = typename Tr::elem;
    using frag = typename Tr::frag;
    constexpr int kpad = KS * Tr::KSTEP;
    constexpr int CAP = WAVE * E;
    constexpr int DEPTH = TREE_DEPTH;
    __shared__ uint64_t s_buf[TNQ][TBUF];
    __shared__ __attribute__((aligned(16))) float s_tau[TNQ];   // score thresholds (-inf: no query)
    __shared__ float s_yq[TNQ], s_box[2 * PR_DIMS];
    const int count = *crv.wide_count;
    if (static_cast<int>(blockIdx.x) >= count) return;
    const int lane = lane_id();
    const int half = lane >> 5, l31 = lane & 31;
    const int t0 = crv.wide[xcd_index(blockIdx.x, count)];
    const int q0 = t0 * TNQ;
    const int nq_valid = min(TNQ, n - q0);
    const int ntiles = crv.layout.cnt[0];
    uint64_t* lists_q0 = lists + static_cast<size_t>(q0) * CAP;
    frag qa[KS];
    {
        const elem* src = Aq + static_cast<size_t>(min(q0 + l31, n - 1)) * kpad + half * Tr::VEC;
#pragma unroll
        for (int s = 0; s < KS; ++s) qa[s] = Tr::load(src + s * Tr::KSTEP);
    }
    const float R = __uint_as_float(*rmax_bits);
    BoxBound bb;
    bb.zerr = crv.zcoef * R;
    bb.pscale = *crv.pscale;
    bb.yerr = crv.ycoef * R;
    PointTest pt;
    {
        const float4 z = reinterpret_cast<const float4*>(crv.zs + static_cast<size_t>(min(q0 + l31, n - 1)) * PR_DIMS)[half];
        pt.z[0] = z.x;
        pt.z[1] = z.y;
        pt.z[2] = z.z;
        pt.z[3] = z.w;
    }
    if (lane < 2 * PR_DIMS) s_box[lane] = crv.tbox[static_cast<size_t>(t0) * 2 * PR_DIMS + lane];
    if (lane < TNQ) {
        s_yq[lane] = lane < nq_valid ? ynorm2[q0 + lane] : 0.f;
        s_tau[lane] = lane < nq_valid ? lb_out[q0 + lane] : -TINF;
    }
    for (int q = 0; q < nq_valid; ++q)
#pragma unroll
        for (int s = 0; s < E; ++s) lists_q0[static_cast<size_t>(q) * CAP + s * WAVE + lane] = KEY_INF;
    wave_lds_sync();
    wave_global_sync();
    auto reach_threshold = [&]() {
        const float t = l31 < nq_valid ? fmaxf(s_tau[l31] + s_yq[l31], 0.f) * (1.f + 4.8e-7f) : -TINF;
        const float p = (sqrtf(fmaxf(t, 0.f)) * (1.f + 1e-6f) + bb.yerr) / bb.pscale + 2.f * 2.8285f * bb.zerr;
        pt.gt = l31 < nq_valid ? p * p * (1.f + 4e-6f) : -TINF;
        return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(wave_max_f32(t))));
    };
    float wthr = reach_threshold();
    float tauv[16];   // this lane's accumulator register r holds row acc_row(r, half)
#pragma unroll
    for (int r = 0; r < 16; ++r) tauv[r] = s_tau[acc_row(r, half)];
    // the buffers' fill, wave-uniform: query q's count in byte q % 4 of cntw[q / 4]
    uint32_t cntw[TNQ / 4];
#pragma unroll
    for (int i = 0; i < TNQ / 4; ++i) cntw[i] = 0u;
    auto cnt_of = [&](int q) { return static_cast<int>((cntw[q >> 2] >> (8 * (q & 3))) & 0xFFu); };

    const int ngroups = (ntiles + WAVE - 1) / WAVE;
    int grp = t0 / WAVE, left = ngroups;   // the next group, groups not yet taken
    int base = 0;
    uint64_t mask = 0ull;
    const bool test = crv.wide_count[1] < TREACH;   // against the single queries too
    auto next_tile = [&]() -> int {
        while (true) {
            if (!mask) {
                if (left == 0) return -1;
                --left;
                base = grp * WAVE;
                grp = grp + 1 == ngroups ? 0 : grp + 1;
                const int v = base + lane;
                float b[2 * PR_DIMS], qb[2 * PR_DIMS];
                load_box(crv.tbox + static_cast<size_t>(min(v, ntiles - 1)) * 2 * PR_DIMS, b);
#pragma unroll
                for (int c = 0; c < 2 * PR_DIMS; ++c) qb[c] = s_box[c];
                mask = __ballot(v < ntiles && box_bound(b, qb, qb + PR_DIMS, bb) <= wthr);
                continue;
            }
            const int c = __builtin_ctzll(mask);
            mask &= mask - 1;
            if (test) {
                const float4* nb = reinterpret_cast<const float4*>(crv.tbox + static_cast<size_t>(base + c) * 2 * PR_DIMS);
                if (!pt.reach(nb[half], nb[PR_DIMS / 4 + half])) continue;
            }
            return base + c;
        }
    };
    int tq[DEPTH];
    frag bq[DEPTH][KS];
    auto load_tile = [&](int t, frag (&b)[KS]) {
        const elem* src = Bc + static_cast<size_t>(max(t, 0)) * 32 * kpad + lane * Tr::VEC;
#pragma unroll
        for (int s = 0; s < KS; ++s) b[s] = Tr::load(src + s * 64 * Tr::VEC);
    };
#pragma unroll
    for (int d = 0; d + 1 < DEPTH; ++d) {
        tq[d] = next_tile();
        load_tile(tq[d], bq[d]);
    }
    unsigned long long pairs = 0;
    bool fell = false;
    while (tq[0] >= 0) {
        if (fell) {
            wthr = reach_threshold();
            fell = false;
        }
        tq[DEPTH - 1] = next_tile();
        load_tile(tq[DEPTH - 1], bq[DEPTH - 1]);
        f32x16 acc = {};
#pragma unroll
        for (int s = 0; s < KS; ++s) acc = Tr::mma(qa[s], bq[0][s], acc);
        const int cand = tq[0] * 32 + l31;
        const bool valid = cand < n;
        pairs += static_cast<unsigned long long>(nq_valid) * __popcll(__ballot(valid) & 0xFFFFFFFFull);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            uint64_t hit = __ballot(valid && acc[r] <= tauv[r]);
            if (!hit) continue;
            const int qa_ = acc_row(r, 0), qb_ = acc_row(r, 1);
            int ca = cnt_of(qa_), cb = cnt_of(qb_);
            const bool fa = ca + __popc(static_cast<uint32_t>(hit)) > TBUF;
            const bool fb = cb + __popc(static_cast<uint32_t>(hit >> 32)) > TBUF;
            if (fa || fb) {
                wave_lds_sync();
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (!(h ? fb : fa)) continue;
                    const int q = h ? qb_ : qa_;
                    const float nt = merge_query_list<E>(lists_q0 + static_cast<size_t>(q) * CAP, &s_buf[q][0],
                                                         h ? cb : ca, kp);
                    if (half == h) tauv[r] = fminf(tauv[r], nt);
                    if (lane == 0) s_tau[q] = fminf(s_tau[q], nt);
                    (h ? cb : ca) = 0;
                    cntw[q >> 2] &= ~(0xFFu << (8 * (q & 3)));
                }
                fell = true;
                wave_lds_sync();
                hit = __ballot(valid && acc[r] <= tauv[r]);
            }
            const int pa = __popc(static_cast<uint32_t>(hit)), pb = __popc(static_cast<uint32_t>(hit >> 32));
            // (mbcnt64 counts the lower half's lanes too in the upper half)
            const int slot0 = half ? qb_ * TBUF + cb - pa : qa_ * TBUF + ca;
            if (valid && acc[r] <= tauv[r])
                (&s_buf[0][0])[slot0 + mbcnt64(hit)] = make_key(acc[r], static_cast<uint32_t>(cand));
            cntw[qa_ >> 2] += static_cast<uint32_t>(pa) << (8 * (qa_ & 3));
            cntw[qb_ >> 2] += static_cast<uint32_t>(pb) << (8 * (qb_ & 3));
        }
#pragma unroll
        for (int d = 0; d + 1 < DEPTH; ++d) {
            tq[d] = tq[d + 1];
#pragma unroll
            for (int s = 0; s < KS; ++s) bq[d][s] = bq[d + 1][s];
        }
    }
    wave_lds_sync();
    int cnt_lane = 0;   // query q's count moved to lane q
#pragma unroll
    for (int q = 0; q < TNQ; ++q)
        if (lane == q) cnt_lane = cnt_of(q);
    for (int q = 0; q < nq_valid; ++q) {
        const float nt = merge_query_list<E>(lists_q0 + static_cast<size_t>(q) * CAP, &s_buf[q][0],
                                             __builtin_amdgcn_readlane(cnt_lane, q), kp);
        if (lane == 0) s_tau[q] = fminf(s_tau[q], nt);
    }
    wave_lds_sync();
    count_pairs(pair_count, pairs);
    if (lane < nq_valid) lb_out[q0 + lane] = certificate_bound(s_tau[lane], s_yq[lane], R, em);
}

// ------------------------------------------------------------------ launcher
struct TreeCall {
    const void *Aq, *Bc;
    int n, kp;
    const float* ynorm2;
    const unsigned* rmax;
    ErrModel em;
    uint64_t* lists;
    int cap;
    float* lb;
    CurveArgs crv;
    unsigned long long* pairs;
    hipStream_t st;
};

// The launchers of ks K-steps; hipErrorNotSupported: not compiled in that file.
hipError_t tree_f32(int ks, const TreeCall& c);        // up to 32
hipError_t tree_f32_wide(int ks, const TreeCall& c);
hipError_t tree_bf16(int ks, const TreeCall& c);       // up to 10
hipError_t tree_bf16_wide(int ks, const TreeCall& c);

// long contractions: the query operand in LDS, the pairwise projected bound
constexpr bool tree_long(int split, int ks) { return ks > (split == 0 ? 16 : 5); }

// Query tiles are handed over where the sampled reach (k_select_tree) exceeds
// this. Short contractions, to k_select_scan: where some 2048 tiles and a
// sixteenth of all are within a query tile's reach (Gaussian n = 100k m = 16
// 15.2 to 10.5 ms; 12-dimensional clusters n = 1M, a tenth within reach, 109 to 78;
// 5-dimensional Gaussian n = 100k, 1200 tiles, 4.2 by the walk and 4.7; the mixture n =
// 8M, one tile in 60, 98 and 125). Long ones, to the workgroup scan of every tile: where
// every sampled tile is (Gaussian n = 100k m = 128 BF16 45 to 20 ms; 7-dimensional
// Gaussian n = 30k m = 64, 99% of them, 3.9 by the walk and 4.6) and the query tiles
// fill the chip (Gaussian n = 8000 m = 64 BF16 2.4 and 2.9; n = 30k 5.7 and 5.0).
constexpr int tree_wide_min(bool is_long, int ntiles)
{
    if (is_long) return ntiles > 512 ? TREACH - 1 : TREACH;
    if (ntiles <= 2048) return TREACH;
    const int share = static_cast<int>(int64_t(2048) * TREACH / ntiles);
    return share > TREACH / 16 ? share : TREACH / 16;
}

template <class Tr, int KS>
static hipError_t launch_tree(const TreeCall& c)
{
    using elem = typename Tr::elem;
    constexpr bool LONG = tree_long(std::is_same<Tr, TraitsF32>::value ? 0 : 3, KS);
    const int n = c.n, kp = c.kp, cap = c.cap;
    if (kp > cap || (cap != 128 && cap != 256)) return hipErrorInvalidValue;
    const int ntiles = (n + 31) / 32;
    if (c.crv.layout.cnt[0] != ntiles) return hipErrorInvalidValue;
    const dim3 grid(ntiles), block(WAVE);
    const elem* A = static_cast<const elem*>(c.Aq);
    const elem* B = static_cast<const elem*>(c.Bc);
    // scores kept per lane and query: the mean share of the kp nearest is kp /
    // 32. Two wavefronts per SIMD, or one where the kept scores, or the query
    // operand in LDS, leave no room for two (then the products' loads run ahead).
    constexpr int W5 = LONG && KS * sizeof(typename Tr::frag) > 13 * 16 ? 1 : 2, W8 = LONG ? 1 : 2;
    const int wide_min = tree_wide_min(LONG, ntiles);
    auto go = [&](auto kernel, bool buf) {
        const size_t keys = buf ? TNQ * TBUF * sizeof(uint64_t) + TNQ * sizeof(int) : 2 * TNQ * sizeof(uint64_t);
        const size_t dyn = tree_operand_bytes<Tr, KS, LONG>() + keys;
        auto run = [&](dim3 g, int probe) {
            hipLaunchKernelGGL(kernel, g, block, dyn, c.st, A, B, n, kp, c.ynorm2, c.rmax, c.em, c.lists, c.lb, c.crv,
                               probe, wide_min, c.pairs);
        };
        if (wide_min < TREACH) run(dim3(WAVE), 1);
        run(grid, 0);
    };
    if (kp <= 96)
        go(k_select_tree<Tr, KS, LONG, 2, 5, false, W5>, false);
    else if (cap == 128)
        go(k_select_tree<Tr, KS, LONG, 2, 8, true, W8>, true);
    else if (kp <= 224)
        go(k_select_tree<Tr, KS, LONG, 4, 8, false, W8>, false);
    else
        go(k_select_tree<Tr, KS, LONG, 4, 12, true, 1>, true);
    if constexpr (!LONG) {   // (the long ones: launch_select_tree)
        auto scan = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, block, 0, c.st, A, B, n, kp, c.ynorm2, c.rmax, c.em, c.lists, c.lb, c.crv,
                               c.pairs);
        };
        if (wide_min < TREACH && cap == 128)
            scan(k_select_scan<Tr, KS, 2>);
        else if (wide_min < TREACH)
            scan(k_select_scan<Tr, KS, 4>);
    }
    return hipGetLastError();
}

}  // namespace kvb
