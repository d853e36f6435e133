// Exact k-nearest-neighbour kernels (gfx950).
//
// The method needs, for every sample, its k-1 nearest other samples in the
// order I(x, k) of Section 2.1 (ties to the smaller index); this fixes the
// sparsity pattern of every kernel matrix in Sections 2.1-2.2. The paper's
// brute-force construction (Section 4, Algorithm 1) evaluates all n^2 pairs;
// its rows are independent, which is the parallelism used here.
//
// Pipeline of kvb_knn for one row i:
//   select   stream all n candidates through a distance test and keep the
//            k' = k + margin smallest (distance, index) keys (one wavefront
//            owns R rows; lanes hold candidates);
//   refine   recompute the k' candidates' squared distances in float64
//            (rounded to float32), drop i itself, sort, decide membership at the
//            k-th neighbour in float64, and check a certificate that no
//            dropped candidate can be nearer than the k-th kept one;
//   fallback rows without a certificate are recomputed by an exact float64
//            radix selection over all n samples.
#include <algorithm>

#include "kvb_device.h"
#include "kvb_kernels.h"

namespace kvb {

// -------------------------------------------------------------------- select
// Direct-difference distance tiles for small m (VALU: m subtractions and m
// multiply-adds per pair; the query coordinates are wave-uniform).
//
// The samples are visited in a spatial order: sorted along a Morton (Z-order)
// curve of their coordinates, cut into tiles of 64 consecutive samples (one
// candidate per lane) and superblocks of 16 tiles, each with its axis-aligned
// bounding box. A wavefront owns R consecutive sorted rows. It first scores
// its own tile and the nearest tiles along the curve, which sets tight
// thresholds, then tests every superblock box (64 per instruction, one per
// lane) and, inside the superblocks within reach, every tile box (16 lanes),
// and scores only the tiles whose box lies within some row's current
// threshold of that row's point. A candidate skipped for a row is therefore at
// least as far as that row's threshold, which only decreases afterwards; this
// keeps the certificate of
// the refine step valid: the box bound is computed in float32 with at most
// (m + 2) roundings, inside the relative margin the refine step allows for
// the selection scores.
//
// Candidates passing the current threshold of a row are appended to that row's
// buffer in LDS, larger than the list's capacity of 64 E keys. When it is full
// (CutRule), bisection over the scores finds a threshold that between kp and 64 E
// of the keys do not exceed; the keys beyond it are dropped and the row's threshold
// is lowered to it. At the end the buffer, cut down in the same way, is sorted
// once. (Merging every 64 keys into a sorted list took three to five networks per
// row where one is enough: 64 nearest of 100k on the torus, 226 to 170 us.) Keys
// carry curve positions; the re-rank maps them to original indices and breaks ties
// on those, so ties order as in I(x, k).
struct SpatialView {
    const float* Xs;      // [n, m] coordinates in curve order
    const float* tbox;    // [tiles, 2, m]: lower corner, then upper corner
    const float* sbox;    // [superblocks, 2, m]
};

constexpr int TILE = 64;
constexpr int SB_TILES = 16;

// Whether a box may hold a candidate for any of the wavefront's rows: the
// squared gap from row r's point to the box against row r's own threshold.
// (Testing the rows' common bounding box instead lets a wavefront whose rows
// straddle a jump of the curve scan far too many tiles.)
template <int M, int R>
__device__ __forceinline__ bool box_near_rows(const float* __restrict__ b, const float (&q)[R][M],
                                              const float (&tau)[R])
{
    float lo[M], hi[M];
#pragma unroll
    for (int c = 0; c < M; ++c) {
        lo[c] = b[c];
        hi[c] = b[M + c];
    }
    bool near = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float s = 0.f;
#pragma unroll
        for (int c = 0; c < M; ++c) {
            const float g = fmaxf(fmaxf(lo[c] - q[r][c], q[r][c] - hi[c]), 0.f);
            s = fmaf(g, g, s);
        }
        near = near || s <= tau[r];
    }
    return near;
}

constexpr int SEED_TILES = 3;   // curve neighbours on each side scored before any box test
constexpr int TILE_BATCH = 2;   // tiles of a superblock whose loads are in flight together

// Upper bound on the kp-th smallest of the wavefront's NS x 64 non-negative
// values (+inf marks none): bisection on the float bit pattern down to bit
// 18 (a relative resolution of 2^-5), by ballot counts; +inf when fewer
// than kp values are finite.
template <int NS>
__device__ __forceinline__ float seed_threshold(const float (&d)[NS], int kp)
{
    int total = 0;
#pragma unroll
    for (int u = 0; u < NS; ++u) total += __popcll(__ballot(d[u] < __uint_as_float(0x7F800000u)));
    if (total < kp) return __uint_as_float(0x7F800000u);
    uint32_t P = 0;
    for (int b = 30; b >= 18; --b) {
        const uint32_t cand = P | (1u << b);
        int cnt = 0;
#pragma unroll
        for (int u = 0; u < NS; ++u) cnt += __popcll(__ballot(__float_as_uint(d[u]) < cand));
        if (cnt < kp) P = cand;
    }
    return __uint_as_float(P | ((1u << 18) - 1u));
}

template <int M>
__device__ __forceinline__ void load_tile(const SpatialView& sv, int n, int t, int lane, float (&x)[M], uint32_t& jo)
{
    const int jp = min(t * TILE + lane, n - 1);
#pragma unroll
    for (int c = 0; c < M; ++c) x[c] = sv.Xs[static_cast<size_t>(jp) * M + c];
    jo = static_cast<uint32_t>(jp);   // curve position; the refine step maps it to the sample id
}

template <int M>
__device__ __forceinline__ float pair_dist2(const float (&q)[M], const float (&x)[M])
{
    float tt = q[0] - x[0];
    float d = tt * tt;
#pragma unroll
    for (int c = 1; c < M; ++c) {
        tt = q[c] - x[c];
        d = fmaf(tt, tt, d);
    }
    return d;
}

// Append the lanes' keys whose score does not exceed tau to a row's buffer
// (which has room for them). Whole wavefront.
__device__ __forceinline__ void append_keys(uint64_t* buf, int& count, float tau, float d, uint32_t j, bool valid)
{
    const bool in = valid && d <= tau;
    const uint64_t mask = __ballot(in);
    if (!mask) return;
    if (in) buf[count + mbcnt64(mask)] = make_key(d, j);
    count += __popcll(mask);
}

// When a row's buffer is cut and how far. Up to five coordinates a row's
// candidates come from few tiles and a cut costs more than a loose threshold: the
// buffer is filled (twice the capacity; 256 keys for lists of 64, which a buffer of
// 128 cut at every further key where kp is 64). From six on the tiles within reach
// grow steeply with the threshold: it is lowered after every 32 further keys (64
// where the threshold has to be close to exact), and the smaller buffer leaves
// room for more wavefronts. Eight coordinates, Gaussian n = 300k: k = 16 19.3 to 16.4
// ms, k = 160 35.3 to 28.1 (16.1 and 25.5 by merges); six, n = 100k, k = 160 3.19 to 2.59.
template <int M, int E>
struct CutRule {
    static constexpr int CAP = WAVE * E;   // of a list
    static constexpr int BUF = M >= 6 ? CAP + 2 * WAVE : E == 1 ? 4 * WAVE : 2 * CAP;
    static constexpr int S = BUF / WAVE;   // keys per lane
    __device__ static int full(int kp)     // cut a buffer of more keys than this (a tile adds up to 64)
    {
        return M >= 6 ? kp + (kp + 32 <= CAP ? 32 : 64) : BUF - WAVE;
    }
    __device__ static int keep(int kp) { return M >= 6 ? min(kp + 8, CAP) : CAP; }   // to at most this many
};

// The 64 E smallest of more keys than a threshold can part (hundreds of equal
// scores), sorted, at the front of the buffer. Whole wavefront. (An LDS pointer:
// through a generic one the stores would not be ordered with the caller's LDS
// reads.)
using lds_key = __attribute__((address_space(3))) uint64_t;
template <int E, int S>
__device__ __noinline__ void sort_front(lds_key* buf, int count)
{
    constexpr int P = S <= 4 ? 4 : 8;   // the network's power of two
    const int lane = lane_id();
    uint64_t v[P];
#pragma unroll
    for (int s = 0; s < P; ++s) v[s] = s < S && s * WAVE + lane < count ? buf[s * WAVE + lane] : KEY_INF;
    bitonic_sort<P>(v);
    wave_lds_sync();
#pragma unroll
    for (int s = 0; s < E; ++s) buf[s * WAVE + lane] = v[s];
    wave_lds_sync();
}

// Drop the farthest of a buffer's count keys (most < count <= 64 S) until
// between kp and `most` are left, which hold the kp smallest; no score above the
// new tau is among the kp smallest. Whole wavefront.
template <int E, int S>
__device__ __forceinline__ void cut_buffer(uint64_t* buf, int& count, float& tau, int kp, int most)
{
    const int lane = lane_id();
    wave_lds_sync();
    uint64_t v[S];
    float d[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
        v[s] = s * WAVE + lane < count ? buf[s * WAVE + lane] : KEY_INF;
        d[s] = key_dist(v[s]);   // +inf past the end: above every threshold tried
    }
    // lo: fewer than kp scores do not exceed it; hi: at least kp do not
    // (scores are >= 0: their bits order like integers)
    uint32_t lo = 0u, hi = __builtin_amdgcn_readfirstlane(__float_as_uint(tau));
    int at = count, below = 0;
    bool parted = false;
    for (int it = 0;; ++it) {
        const float a = __uint_as_float(lo), b = __uint_as_float(hi);
        // twice where the counts' share falls, then the middle; where neither
        // lies inside (infinite or adjacent ends), the middle of the bits
        const float share = it < 2 ? static_cast<float>((kp + most) / 2 - below) *
                                         __builtin_amdgcn_rcpf(static_cast<float>(at - below))
                                   : 0.5f;
        uint32_t mid = __builtin_amdgcn_readfirstlane(__float_as_uint(fmaf(share, b - a, a)));
        if (!(mid > lo && mid < hi)) mid = lo + (hi - lo) / 2;
        if (mid == lo) break;
        int c = 0;
#pragma unroll
        for (int s = 0; s < S; ++s) c += __popcll(__ballot(d[s] <= __uint_as_float(mid)));
        if (c < kp) {
            lo = mid;
            below = c;
        } else {
            hi = mid;
            at = c;
            if (c <= most) {
                parted = true;
                break;
            }
        }
    }
    if (parted) {
        const float thr = __uint_as_float(hi);
        int w = 0;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const bool in = d[s] <= thr;
            const uint64_t mask = __ballot(in);
            if (in) buf[w + mbcnt64(mask)] = v[s];
            w += __popcll(mask);
        }
        tau = thr;
        count = at;
        wave_lds_sync();
    } else {
        sort_front<E, S>((lds_key*)buf, count);
        count = min(count, most);
        tau = fminf(tau, key_dist(buf[kp - 1]));
    }
}

template <int M, int R, int E>
__global__ __launch_bounds__(256) void k_select_direct(SpatialView sv, int n, int kp,
                                                       uint64_t* __restrict__ keys_out,
                                                       float* __restrict__ slast_out,
                                                       unsigned long long* __restrict__ pair_count)
{
    using Cut = CutRule<M, E>;
    constexpr int CAP = Cut::CAP, BUF = Cut::BUF;
    const int full = Cut::full(kp), keep = Cut::keep(kp);
    __shared__ uint64_t sbuf[4][R][BUF];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row0 = (blockIdx.x * 4 + wave) * R;   // curve position of the first row
    if (row0 >= n) return;

    float q[R][M];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int p = min(row0 + r, n - 1);
#pragma unroll
        for (int c = 0; c < M; ++c) q[r][c] = sv.Xs[static_cast<size_t>(p) * M + c];
    }
    float tau[R];
    int bc[R];
    const int rows_here = min(R, n - row0);
    unsigned long long pairs = 0;

    const int ntiles = (n + TILE - 1) / TILE;
    const int nsb = (ntiles + SB_TILES - 1) / SB_TILES;
    const int own_t = row0 / TILE;
    // the tiles base + t, t a bit of tm: their loads issued TILE_BATCH at a time
    auto scan_tiles = [&](int base, uint64_t tm) {
        while (tm) {
            int tb[TILE_BATCH];
            float xb[TILE_BATCH][M];
            uint32_t jb[TILE_BATCH];
#pragma unroll
            for (int u = 0; u < TILE_BATCH; ++u) {
                tb[u] = -1;
                jb[u] = 0;
                if (tm) {
                    tb[u] = base + __builtin_ctzll(tm);
                    tm &= tm - 1;
                    load_tile<M>(sv, n, tb[u], lane, xb[u], jb[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < TILE_BATCH; ++u) {
                if (tb[u] < 0) continue;
                const bool valid = tb[u] * TILE + lane < n;
                pairs += static_cast<unsigned long long>(min(TILE, n - tb[u] * TILE)) * rows_here;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if (bc[r] > full) cut_buffer<E, Cut::S>(sbuf[wave][r], bc[r], tau[r], kp, keep);
                    append_keys(sbuf[wave][r], bc[r], tau[r], pair_dist2<M>(q[r], xb[u]), jb[u], valid);
                }
            }
        }
    };
    // seed: the own tile and its curve neighbours, unconditionally. Each row's
    // first threshold is a coarse upper bound of the kp-th smallest seed
    // distance (valid for the whole scan: the kp-th smallest of a subset is at
    // least the kp-th smallest overall), so the seeds append little more than kp.
    constexpr int NS = 2 * SEED_TILES + 1;
    const int a0 = max(0, own_t - SEED_TILES), a1 = min(ntiles - 1, own_t + SEED_TILES);
    {
        float xs[NS][M];
        uint32_t js[NS];
        bool ok[NS];
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            load_tile<M>(sv, n, min(a0 + u, a1), lane, xs[u], js[u]);
            ok[u] = (a0 + u <= a1) && ((a0 + u) * TILE + lane < n);
        }
        bool fits = true;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float ds[NS];
#pragma unroll
            for (int u = 0; u < NS; ++u) ds[u] = ok[u] ? pair_dist2<M>(q[r], xs[u]) : __uint_as_float(0x7F800000u);
            bc[r] = 0;
            tau[r] = seed_threshold<NS>(ds, kp);
            int c = 0;
#pragma unroll
            for (int u = 0; u < NS; ++u) c += __popcll(__ballot(ok[u] && ds[u] <= tau[r]));
            // more equal scores than the buffer holds: tile by tile below
            fits = fits && c <= BUF;
            if (c <= BUF) {
#pragma unroll
                for (int u = 0; u < NS; ++u)
                    append_keys(sbuf[wave][r], bc[r], tau[r], ds[u], js[u], ok[u]);
            }
        }
        if (fits) {
            pairs += static_cast<unsigned long long>(min(n, (a1 + 1) * TILE) - a0 * TILE) * rows_here;
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) bc[r] = 0;
            wave_lds_sync();
            scan_tiles(a0, (1ull << (a1 - a0 + 1)) - 1ull);
        }
    }
    // then every superblock within reach of some row (boxes tested 64 at a
    // time, one per lane), inside it every tile within reach (16 lanes)
    for (int sb0 = 0; sb0 < nsb; sb0 += WAVE) {
        const int sbl = sb0 + lane;
        bool near = false;
        if (sbl < nsb) near = box_near_rows<M, R>(sv.sbox + static_cast<size_t>(sbl) * 2 * M, q, tau);
        uint64_t sbm = __ballot(near);
        while (sbm) {
            const int sb = sb0 + __builtin_ctzll(sbm);
            sbm &= sbm - 1;
            const int tl = sb * SB_TILES + lane;
            bool tnear = false;
            if (lane < SB_TILES && tl < ntiles && (tl < a0 || tl > a1))
                tnear = box_near_rows<M, R>(sv.tbox + static_cast<size_t>(tl) * 2 * M, q, tau);
            scan_tiles(sb * SB_TILES, __ballot(tnear));
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (bc[r] > CAP) cut_buffer<E, Cut::S>(sbuf[wave][r], bc[r], tau[r], kp, CAP);
        wave_lds_sync();
        if (row0 + r < n) {
            uint64_t L[E];
#pragma unroll
            for (int s = 0; s < E; ++s) L[s] = s * WAVE + lane < bc[r] ? sbuf[wave][r][s * WAVE + lane] : KEY_INF;
            bitonic_sort<E>(L);
            const int i = row0 + r;   // lists are stored by curve position
            uint64_t* dst = keys_out + static_cast<size_t>(i) * kp;
#pragma unroll
            for (int s = 0; s < E; ++s) {
                const int t = s * WAVE + lane;
                if (t < kp) dst[t] = L[s];
            }
            const float sl = key_dist(list_at<E>(L, kp - 1));
            if (lane == 0) slast_out[i] = sl;
        }
    }
    count_pairs(pair_count, pairs);
}

// ---- spatial order of the direct path
// Bounding box of the samples: per-block partial minima / maxima (k_morton
// reduces them). Coordinates together, one barrier: 3 us at 2000 x 3 and 5 at
// 100k x 3 (6 and 14 with a tree of eight barriers per coordinate).
constexpr int BBOX_THREADS = 1024;
template <int M>
__global__ __launch_bounds__(BBOX_THREADS) void k_bbox_partial(const float* __restrict__ X, int n, int rows_per_block,
                                                               float* __restrict__ part)
{
    constexpr int WAVES = BBOX_THREADS / WAVE;
    __shared__ float s_b[WAVES][2 * M];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int r0 = blockIdx.x * rows_per_block, r1 = min(n, r0 + rows_per_block);
    const float inf = __uint_as_float(0x7F800000u);
    float lo[M], hi[M];
#pragma unroll
    for (int c = 0; c < M; ++c) {
        lo[c] = inf;
        hi[c] = -inf;
    }
#pragma unroll 4
    for (int r = r0 + threadIdx.x; r < r1; r += BBOX_THREADS) {
#pragma unroll
        for (int c = 0; c < M; ++c) {
            const float v = X[static_cast<size_t>(r) * M + c];
            lo[c] = fminf(lo[c], v);
            hi[c] = fmaxf(hi[c], v);
        }
    }
#pragma unroll
    for (int c = 0; c < M; ++c) {
#pragma unroll
        for (int o = 1; o < WAVE; o <<= 1) {
            lo[c] = fminf(lo[c], shfl_xor_f32(lo[c], o));
            hi[c] = fmaxf(hi[c], shfl_xor_f32(hi[c], o));
        }
        if (lane == 0) {
            s_b[wave][c] = lo[c];
            s_b[wave][M + c] = hi[c];
        }
    }
    __syncthreads();
    if (threadIdx.x < 2 * M) {
        const int c = threadIdx.x;
        float v = s_b[0][c];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) v = c < M ? fminf(v, s_b[w][c]) : fmaxf(v, s_b[w][c]);
        part[static_cast<size_t>(blockIdx.x) * 2 * M + c] = v;
    }
}

// Morton code of every sample: each coordinate quantised to b = min(31, 32 / m) bits
// over the bounding box (every workgroup reduces the box partials: at most 1024
// of 2m values), bits interleaved from the most significant. value = sample
// index, so a stable sort breaks ties by index.
__global__ __launch_bounds__(256) void k_morton(const float* __restrict__ X, int n, int m, int bits,
                                                const float* __restrict__ part, int nparts,
                                                uint32_t* __restrict__ code, int32_t* __restrict__ vals)
{
    __shared__ float s_lo[8], s_scale[8];
    // a wavefront per coordinate, a partial per lane
    for (int c = threadIdx.x >> 6; c < m; c += 4) {
        float lo = __uint_as_float(0x7F800000u), hi = -__uint_as_float(0x7F800000u);
        for (int b = lane_id(); b < nparts; b += WAVE) {
            lo = fminf(lo, part[static_cast<size_t>(b) * 2 * m + c]);
            hi = fmaxf(hi, part[static_cast<size_t>(b) * 2 * m + m + c]);
        }
#pragma unroll
        for (int o = 1; o < WAVE; o <<= 1) {
            lo = fminf(lo, shfl_xor_f32(lo, o));
            hi = fmaxf(hi, shfl_xor_f32(hi, o));
        }
        if (lane_id() == 0) {
            const float ext = hi - lo;
            s_lo[c] = lo;
            s_scale[c] = ext > 0.f ? static_cast<float>(1ull << bits) / ext : 0.f;
        }
    }
    __syncthreads();
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t qc[8];
    const uint32_t qmax = static_cast<uint32_t>((1ull << bits) - 1);
    for (int c = 0; c < m; ++c) {
        const float t = (X[static_cast<size_t>(i) * m + c] - s_lo[c]) * s_scale[c];
        const float tc = fminf(fmaxf(t, 0.f), static_cast<float>(qmax));
        qc[c] = min(static_cast<uint32_t>(tc), qmax);
    }
    uint32_t z = 0;
    for (int b = bits - 1; b >= 0; --b)
        for (int c = 0; c < m; ++c) z = (z << 1) | ((qc[c] >> b) & 1u);
    code[i] = z;
    vals[i] = i;
}

__global__ __launch_bounds__(256) void k_gather_rows(const float* __restrict__ X, int n, int m,
                                                     const int32_t* __restrict__ perm, float* __restrict__ Xs)
{
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= static_cast<int64_t>(n) * m) return;
    const int p = static_cast<int>(t / m), c = static_cast<int>(t % m);
    Xs[t] = X[static_cast<size_t>(perm[p]) * m + c];
}

// the same with four coordinates per thread (m a multiple of 4, rows 16-byte aligned)
__global__ __launch_bounds__(256) void k_gather_rows4(const float4* __restrict__ X, int n, int m4,
                                                      const int32_t* __restrict__ perm, float4* __restrict__ Xs)
{
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= static_cast<int64_t>(n) * m4) return;
    const int p = static_cast<int>(t / m4), c = static_cast<int>(t % m4);
    Xs[t] = X[static_cast<size_t>(perm[p]) * m4 + c];
}

// Xs[p] = X[perm[p]], float4 pieces where the rows allow
static void gather_rows(const float* X, int n, int m, const int32_t* perm, float* Xs, hipStream_t st)
{
    const bool v4 =
        m % 4 == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0 && (reinterpret_cast<uintptr_t>(Xs) & 15) == 0;
    const int64_t tot = static_cast<int64_t>(n) * (v4 ? m / 4 : m);
    const dim3 grid(static_cast<unsigned>((tot + 255) / 256));
    if (v4)
        hipLaunchKernelGGL(k_gather_rows4, grid, dim3(256), 0, st, reinterpret_cast<const float4*>(X), n, m / 4, perm,
                           reinterpret_cast<float4*>(Xs));
    else
        hipLaunchKernelGGL(k_gather_rows, grid, dim3(256), 0, st, X, n, m, perm, Xs);
}

// Curve-ordered samples, tile boxes and superblock boxes in one launch: a
// workgroup per superblock, a wavefront per tile, a sample per lane: 3 us at
// 2000 x 3 and 5 at 100k x 3 (16 and 19 in three launches of one thread per
// coordinate and box, each reading its rows one after the other).
constexpr int LAYOUT_THREADS = SB_TILES * WAVE;
template <int M>
__global__ __launch_bounds__(LAYOUT_THREADS) void k_spatial_layout(const float* __restrict__ X, int n,
                                                                   const int32_t* __restrict__ perm,
                                                                   float* __restrict__ Xs, float* __restrict__ tbox,
                                                                   float* __restrict__ sbox)
{
    __shared__ float s_lo[SB_TILES][M], s_hi[SB_TILES][M];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = blockIdx.x * SB_TILES + wave;   // tile
    const int p = t * TILE + lane;
    const float inf = __uint_as_float(0x7F800000u);
    float lo[M], hi[M];
#pragma unroll
    for (int c = 0; c < M; ++c) {
        lo[c] = inf;
        hi[c] = -inf;
    }
    if (p < n) {
        const float* x = X + static_cast<size_t>(perm[p]) * M;
#pragma unroll
        for (int c = 0; c < M; ++c) {
            const float v = x[c];
            Xs[static_cast<size_t>(p) * M + c] = v;
            lo[c] = fminf(lo[c], v);
            hi[c] = fmaxf(hi[c], v);
        }
    }
#pragma unroll
    for (int c = 0; c < M; ++c) {
#pragma unroll
        for (int o = 1; o < WAVE; o <<= 1) {
            lo[c] = fminf(lo[c], shfl_xor_f32(lo[c], o));
            hi[c] = fmaxf(hi[c], shfl_xor_f32(hi[c], o));
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int c = 0; c < M; ++c) {
            s_lo[wave][c] = lo[c];
            s_hi[wave][c] = hi[c];
            if (t * TILE < n) {
                tbox[static_cast<size_t>(t) * 2 * M + c] = lo[c];
                tbox[static_cast<size_t>(t) * 2 * M + M + c] = hi[c];
            }
        }
    }
    __syncthreads();
    if (threadIdx.x < M) {
        const int c = threadIdx.x;
        float l = inf, h = -inf;
#pragma unroll
        for (int u = 0; u < SB_TILES; ++u) {   // tiles past the end hold empty boxes
            l = fminf(l, s_lo[u][c]);
            h = fmaxf(h, s_hi[u][c]);
        }
        sbox[static_cast<size_t>(blockIdx.x) * 2 * M + c] = l;
        sbox[static_cast<size_t>(blockIdx.x) * 2 * M + M + c] = h;
    }
}

// -------------------------------------------------------------------- refine
// Squared distances of row a to the rows b_s = B + j_s m (where act_s), each
// accumulated in float64 over the columns in order (the difference of two
// float32 values is exact in float64) and rounded once to float32: the same
// operations as dist2_f64, so these agree bit for bit with the exact path's
// distances. On gfx950 an unpacked float64 FMA issues at the float32 rate,
// so this costs about three instructions per coordinate. The coordinates are
// read CH at a time (float4 pieces when vec4), so that a chunk's loads are in
// flight together.
template <int E, int CH>
__device__ __forceinline__ void dist2_rows_ch(const float* __restrict__ a, const float* __restrict__ B, int m,
                                              const int (&j)[E], const bool (&act)[E], bool vec4, float (&out)[E])
{
    double acc[E];
#pragma unroll
    for (int s = 0; s < E; ++s) acc[s] = 0.0;
    for (int c0 = 0; c0 < m; c0 += CH) {
        float av[CH], bv[E][CH];
        if (vec4) {
#pragma unroll
            for (int u = 0; u < CH / 4; ++u) {
                if (c0 + 4 * u < m) {
                    const float4 q = *reinterpret_cast<const float4*>(a + c0 + 4 * u);
                    av[4 * u] = q.x;
                    av[4 * u + 1] = q.y;
                    av[4 * u + 2] = q.z;
                    av[4 * u + 3] = q.w;
                }
            }
#pragma unroll
            for (int s = 0; s < E; ++s) {
                const float* b = B + static_cast<size_t>(j[s]) * m;
#pragma unroll
                for (int u = 0; u < CH / 4; ++u) {
                    if (act[s] && c0 + 4 * u < m) {
                        const float4 q = *reinterpret_cast<const float4*>(b + c0 + 4 * u);
                        bv[s][4 * u] = q.x;
                        bv[s][4 * u + 1] = q.y;
                        bv[s][4 * u + 2] = q.z;
                        bv[s][4 * u + 3] = q.w;
                    }
                }
            }
        } else {
#pragma unroll
            for (int t = 0; t < CH; ++t)
                if (c0 + t < m) av[t] = a[c0 + t];
#pragma unroll
            for (int s = 0; s < E; ++s) {
                const float* b = B + static_cast<size_t>(j[s]) * m;
#pragma unroll
                for (int t = 0; t < CH; ++t)
                    if (act[s] && c0 + t < m) bv[s][t] = b[c0 + t];
            }
        }
#pragma unroll
        for (int t = 0; t < CH; ++t) {
            if (c0 + t < m) {
#pragma unroll
                for (int s = 0; s < E; ++s)
                    if (act[s]) {
                        const double d = static_cast<double>(av[t]) - static_cast<double>(bv[s][t]);
                        acc[s] = fma(d, d, acc[s]);
                    }
            }
        }
    }
#pragma unroll
    for (int s = 0; s < E; ++s) out[s] = static_cast<float>(acc[s]);
}

// the chunk fitted to m (8 coordinates at most for four key slots)
template <int E>
__device__ __forceinline__ void dist2_rows(const float* __restrict__ a, const float* __restrict__ B, int m,
                                           const int (&j)[E], const bool (&act)[E], bool vec4, float (&out)[E])
{
    if (m <= 4)
        dist2_rows_ch<E, 4>(a, B, m, j, act, vec4, out);
    else if (m <= 8 || E >= 4)
        dist2_rows_ch<E, 8>(a, B, m, j, act, vec4, out);
    else
        dist2_rows_ch<E, 16>(a, B, m, j, act, vec4, out);
}

__device__ __forceinline__ double dist2_f64(const float* __restrict__ a, const float* __restrict__ b, int m)
{
    double s = 0.0;
    for (int c = 0; c < m; ++c) {
        const double t = static_cast<double>(a[c]) - static_cast<double>(b[c]);
        s = fma(t, t, s);
    }
    return s;
}

// Squared distances of a row's candidates computed cooperatively: groups of
// LPC lanes share one candidate (coalesced reads of its row, float4 where the
// rows are 16-byte aligned), accumulate in float64 (differences of float32
// values and their squares are exact or nearly so in float64) and reduce
// inside the group; the result reaches the lane that owns the candidate's key.
// d[s] receives the distance of key slot s of this lane (unchanged where the
// key is KEY_INF or the row itself).
//
// group_distances4: rows of float4 pieces (NIT per lane), two candidates per
// group at a time, their sums reduced together: the first exchange leaves each
// lane one of the two. No load is guarded, so all of a pass are in flight at
// once (behind guards they waited for one another): pieces beyond the row are
// read from zeros. 160 candidates of 128 coordinates per row: 4M rows along the
// curve 38.5 to 21.5 ms, 1M rows by bucket 9.1 to 5.2 (four candidates at a
// time: 21.9 and 5.5).
__device__ const float4 g_zero4 = {0.f, 0.f, 0.f, 0.f};

template <int E, int LPC, int NIT>
__device__ __forceinline__ void group_distances4(const float* __restrict__ X, int m, int i, int kp,
                                                 const uint64_t (&v)[E], double (&d)[E])
{
    constexpr int CPW = WAVE / LPC;   // groups
    constexpr int U = 2;              // candidates per group at a time
    const int lane = lane_id();
    const int g = lane / LPC, gl = lane % LPC;
    bool in[NIT];
    double q[NIT][4];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int c = 4 * (gl + LPC * it);
        in[it] = c < m;
        const float4 t = in[it] ? *reinterpret_cast<const float4*>(X + static_cast<size_t>(i) * m + c) : g_zero4;
        q[it][0] = t.x;
        q[it][1] = t.y;
        q[it][2] = t.z;
        q[it][3] = t.w;
    }
#pragma unroll
    for (int s = 0; s < E; ++s) {
        const int cj = (v[s] != KEY_INF) ? static_cast<int>(key_idx(v[s])) : -1;
        const int tend = min(kp, (s + 1) * WAVE);
        for (int t0 = s * WAVE; t0 < tend; t0 += U * CPW) {
            float4 p[U][NIT];
            bool ok[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                // an invalid slot reads row i and is zeroed
                const int t = t0 + u * CPW;
                const int j = __shfl(cj, (t % WAVE) + g, WAVE);
                ok[u] = j >= 0 && j != i && t + g < tend;
                const float* x = X + static_cast<size_t>(ok[u] ? j : i) * m + 4 * gl;
#pragma unroll
                for (int it = 0; it < NIT; ++it) {
                    const float4* src = in[it] ? reinterpret_cast<const float4*>(x + 4 * LPC * it) : &g_zero4;
                    p[u][it] = *src;
                }
            }
            double acc[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                double a = 0.0;
#pragma unroll
                for (int it = 0; it < NIT; ++it) {
                    const double e0 = q[it][0] - p[u][it].x, e1 = q[it][1] - p[u][it].y;
                    const double e2 = q[it][2] - p[u][it].z, e3 = q[it][3] - p[u][it].w;
                    a = fma(e0, e0, a);
                    a = fma(e1, e1, a);
                    a = fma(e2, e2, a);
                    a = fma(e3, e3, a);
                }
                acc[u] = ok[u] ? a : 0.0;
            }
            // lane gl ends with candidate gl mod 2's sum over the group
            const bool odd = gl & 1;
            double r = (odd ? acc[1] : acc[0]) + shfl_xor_f64(odd ? acc[0] : acc[1], 1);
#pragma unroll
            for (int o = 2; o < LPC; o <<= 1) r += shfl_xor_f64(r, o);
            // to the lanes that own the candidates
            const int at = lane - (t0 % WAVE);
            const bool mine = at >= 0 && at < U * CPW;
            const double got = __shfl(r, mine ? (at % CPW) * LPC + at / CPW : 0, WAVE);
            if (mine) d[s] = got;
        }
    }
}

template <int E, int LPC>
__device__ __forceinline__ void group_distances(const float* __restrict__ X, int m, int i, int kp, bool vec4,
                                                const uint64_t (&v)[E], double (&d)[E])
{
    if (vec4) {
        if (m > 12 * LPC)
            group_distances4<E, LPC, 4>(X, m, i, kp, v, d);
        else
            group_distances4<E, LPC, 3>(X, m, i, kp, v, d);
        return;
    }
    constexpr int CPW = WAVE / LPC;   // candidates per pass
    constexpr int QMAX = 16;          // floats of the row per lane (m <= 16 LPC)
    const int lane = lane_id();
    const int g = lane / LPC, gl = lane % LPC;
    const float* xi = X + static_cast<size_t>(i) * m;
    float q1[QMAX];
    const int nit = (m + LPC - 1) / LPC;
#pragma unroll
    for (int it = 0; it < QMAX; ++it) {
        q1[it] = 0.f;
        if (it < nit) {
            const int c = gl + LPC * it;
            if (c < m) q1[it] = xi[c];
        }
    }
#pragma unroll
    for (int s = 0; s < E; ++s) {
        const int cj = (v[s] != KEY_INF) ? static_cast<int>(key_idx(v[s])) : -1;
        const int tend = min(kp, (s + 1) * WAVE);
        for (int t0 = s * WAVE; t0 < tend; t0 += CPW) {
            const int owner = (t0 % WAVE) + g;                 // lane holding this group's candidate
            const int j = __shfl(cj, owner, WAVE);
            double acc = 0.0;
            if (j >= 0 && j != i && t0 + g < kp) {
                const float* xj = X + static_cast<size_t>(j) * m;
#pragma unroll
                for (int it = 0; it < QMAX; ++it) {
                    const int c = gl + LPC * it;
                    if (it < nit && c < m) {
                        const double e0 = static_cast<double>(q1[it]) - xj[c];
                        acc = fma(e0, e0, acc);
                    }
                }
            }
#pragma unroll
            for (int o = 1; o < LPC; o <<= 1) acc += shfl_xor_f64(acc, o);
            // the group leader's sum goes to the owner lane
            const int src = (lane - (t0 % WAVE)) * LPC;
            const double got = __shfl(acc, src >= 0 && src < WAVE ? src : 0, WAVE);
            if (lane >= t0 % WAVE && lane < t0 % WAVE + CPW) d[s] = got;
        }
    }
}

// One wavefront per row. keys: [n, kstride] candidate keys from a select
// kernel (the first kp of each row are used), slast: per row, a bound on the
// candidates the select step dropped, turned into a lower bound on their true
// squared distance by lb_scale (direct tiles: the kp-th score times
// 1/(1 + select error); matrix-core tiles: the bound itself, lb_scale = 1).
// slast == nullptr: no bound (learned routing). LPC == 0: each lane computes
// its own candidates' distances (float64 sums rounded to float32, short rows);
// LPC > 0: groups of LPC lanes per candidate (group_distances, long rows).
// Lists whose recomputed keys are still in ascending order once row i is taken
// out (the common case after the direct tiles, whose float32 scores differ
// from the recomputed distances only in the last bits) skip the sorting
// network.
//
// Rows are taken in the order of the workgroups' XCDs (xcd_block): the rows in
// flight on an XCD are neighbours along the curve or, with `order` (learned
// routing: the samples grouped by their first bucket), of one bucket, and find
// each other's candidates in its L2 (1M rows by bucket 13.5 to 9.1 ms).
//
// CV (curve-ordered scans): lists and bounds are stored by curve position r, their
// keys hold curve positions; the candidates are read from the curve-ordered
// copy Xs (neighbouring rows read neighbouring samples) and the keys are
// turned into (distance, sample id) through perm before any ordering.
template <int E, int LPC, bool CV>
__global__ __launch_bounds__(256) void k_refine(const float* __restrict__ X, int n, int m, int k, int kp,
                                                int kstride, const uint64_t* __restrict__ keys,
                                                const float* __restrict__ slast, float lb_scale,
                                                int32_t* __restrict__ idx_out, float* __restrict__ d2_out,
                                                int32_t* __restrict__ flags_out,
                                                int* __restrict__ fb_count, int* __restrict__ fb_list,
                                                float* __restrict__ fb_bound, int force_period,
                                                const float* __restrict__ Xs, const int32_t* __restrict__ perm,
                                                const int32_t* __restrict__ order)
{
    const int lane = lane_id();
    const int p = xcd_block() * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (p >= n) return;
    const int r = !CV && order ? order[p] : p;   // stored row
    const int i = CV ? perm[r] : r;   // sample id
    const float* xi = CV ? Xs + static_cast<size_t>(r) * m : X + static_cast<size_t>(i) * m;
    // candidate distances, self removed
    uint64_t v[E];
#pragma unroll
    for (int s = 0; s < E; ++s) {
        const int t = s * WAVE + lane;
        v[s] = t < kp ? keys[static_cast<size_t>(r) * kstride + t] : KEY_INF;
    }
    // list position of row i, if present
    int ps = -1;
#pragma unroll
    for (int s = 0; s < E; ++s) {
        const uint64_t mm = __ballot(v[s] != KEY_INF && static_cast<int>(key_idx(v[s])) == r);
        if (ps < 0 && mm) ps = s * WAVE + __builtin_ctzll(mm);
    }
    if constexpr (LPC == 0) {
        int jr[E];
        bool act[E];
#pragma unroll
        for (int s = 0; s < E; ++s) {
            act[s] = v[s] != KEY_INF && static_cast<int>(key_idx(v[s])) != r;
            jr[s] = act[s] ? static_cast<int>(key_idx(v[s])) : 0;
        }
        const float* Br = CV ? Xs : X;   // the rows the keys refer to
        const bool vec4 = (m % 4 == 0) && ((reinterpret_cast<uintptr_t>(Br) & 15) == 0);
        float dd[E];
        dist2_rows<E>(xi, Br, m, jr, act, vec4, dd);
#pragma unroll
        for (int s = 0; s < E; ++s) {
            if (v[s] == KEY_INF) continue;
            if (!act[s])
                v[s] = KEY_INF;
            else if constexpr (CV)
                v[s] = make_key(dd[s], static_cast<uint32_t>(perm[jr[s]]));
            else
                v[s] = make_key(dd[s], static_cast<uint32_t>(jr[s]));
        }
    } else {
        double dd[E];
#pragma unroll
        for (int s = 0; s < E; ++s) dd[s] = 0.0;
        const float* Xr = CV ? Xs : X;   // the rows the keys refer to
        const bool vec4 = (m % 4 == 0) && ((reinterpret_cast<uintptr_t>(Xr) & 15) == 0);
        group_distances<E, LPC>(Xr, m, r, kp, vec4, v, dd);
#pragma unroll
        for (int s = 0; s < E; ++s) {
            uint64_t key = v[s];
            if (key != KEY_INF) {
                const uint32_t j = key_idx(key);
                key = static_cast<int>(j) == r
                          ? KEY_INF
                          : make_key(static_cast<float>(dd[s]), CV ? static_cast<uint32_t>(perm[j]) : j);
            }
            v[s] = key;
        }
    }
    {
        // the keys one position on, with row i (now KEY_INF) moved past the end
        uint64_t nv[E];
        bool sorted = true;
#pragma unroll
        for (int s = 0; s < E; ++s) {
            uint64_t nx = shfl_u64(v[s], (lane + 1) & (WAVE - 1));
            if (lane == WAVE - 1) nx = (s + 1 < E) ? readlane_u64(v[s + 1 < E ? s + 1 : s], 0) : KEY_INF;
            nv[s] = (ps >= 0 && s * WAVE + lane >= ps) ? nx : v[s];
        }
#pragma unroll
        for (int s = 0; s < E; ++s) {
            uint64_t nx = shfl_u64(nv[s], (lane + 1) & (WAVE - 1));
            if (lane == WAVE - 1) nx = (s + 1 < E) ? readlane_u64(nv[s + 1 < E ? s + 1 : s], 0) : KEY_INF;
            sorted = sorted && !__ballot(nv[s] > nx);
        }
        if (sorted) {
#pragma unroll
            for (int s = 0; s < E; ++s) v[s] = nv[s];
        } else {
            bitonic_sort<E>(v);
        }
    }

    const int kk = k - 1;  // neighbours other than i
    int32_t* orow = idx_out + static_cast<size_t>(i) * k;
    float* drow = d2_out + static_cast<size_t>(i) * k;
    if (lane == 0) {
        orow[0] = i;
        drow[0] = 0.f;
    }
    int flags = 0;
    bool certified = true;
    float bound = __uint_as_float(0x7F800000u);   // upper bound on the true (k-1)-th distance
    if (kk > 0) {
        // relative error bound of the recomputed distances (a few units in
        // the last place), doubled for the band test
        const float dl = 4.8e-7f;
        const float a = key_dist(list_at<E>(v, kk - 1));
        const float lo_edge = a * (1.f - dl) / (1.f + dl);
        const float hi_edge = a * (1.f + dl) / (1.f - dl);
        // positions: sure-in (below lo_edge), band, sure-out (above hi_edge)
        uint64_t band_m[E];
        int c_lo = 0, nband = 0, band_beyond = 0, nvalid = 0;
#pragma unroll
        for (int s = 0; s < E; ++s) {
            const int t = s * WAVE + lane;
            const float dv = key_dist(v[s]);
            const bool valid = v[s] != KEY_INF;
            nvalid += __popcll(__ballot(valid));
            const bool in_lo = valid && dv < lo_edge;
            const bool in_band = valid && !in_lo && dv <= hi_edge;
            c_lo += __popcll(__ballot(in_lo));
            band_m[s] = __ballot(in_band);
            nband += __popcll(band_m[s]);
            band_beyond += __popcll(__ballot(in_band && t >= kk));
        }
        // FP64 recheck only when the band straddles the k-th position
        double d64[E];
        int rank[E];
#pragma unroll
        for (int s = 0; s < E; ++s) {
            d64[s] = 0.0;
            rank[s] = 0;
        }
        const bool recheck = band_beyond > 0;
        if (recheck) {
            flags |= KVB_ROW_RECHECK;
#pragma unroll
            for (int s = 0; s < E; ++s)
                if ((band_m[s] >> lane) & 1ull)
                    d64[s] = dist2_f64(xi, X + static_cast<size_t>(key_idx(v[s])) * m, m);
            // rank of every band member among band members by (d64, j)
#pragma unroll
            for (int so = 0; so < E; ++so) {
                uint64_t bm = band_m[so];
                while (bm) {
                    const int src = __builtin_ctzll(bm);
                    bm &= bm - 1;
                    const double od = __shfl(d64[so], src, WAVE);
                    const uint32_t oj = __builtin_amdgcn_readlane(static_cast<int>(key_idx(v[so])), src);
#pragma unroll
                    for (int s = 0; s < E; ++s) {
                        const uint32_t mj = key_idx(v[s]);
                        if ((od < d64[s]) || (od == d64[s] && oj < mj)) rank[s]++;
                    }
                }
            }
        }
        // write the k-1 neighbours and find the largest kept distance
        float kept_max = 0.f;
        int nkept = 0;
        const int need = kk - c_lo;
#pragma unroll
        for (int s = 0; s < E; ++s) {
            const int t = s * WAVE + lane;
            const bool valid = v[s] != KEY_INF;
            const float dv = key_dist(v[s]);
            const bool in_lo = valid && dv < lo_edge;
            const bool in_band = (band_m[s] >> lane) & 1ull;
            int pos = -1;
            float outd = dv;
            if (in_lo) {
                pos = t;
            } else if (in_band) {
                if (recheck) {
                    if (rank[s] < need) {
                        pos = c_lo + rank[s];
                        outd = static_cast<float>(d64[s]);
                    }
                } else if (t < kk) {
                    pos = t;
                }
            }
            if (pos >= 0) {
                orow[1 + pos] = static_cast<int32_t>(key_idx(v[s]));
                drow[1 + pos] = outd;
                kept_max = fmaxf(kept_max, dv);
            }
            nkept += __popcll(__ballot(pos >= 0));
        }
        kept_max = wave_max_f32(kept_max);
        // the kept candidates are k-1 samples within this distance of row i
        if (nkept == kk) bound = kept_max * (1.f + dl) * (1.f + 1e-6f);
        if (slast) {
            // certificate: every candidate the select step dropped has a true
            // squared distance >= slast * lb_scale; it must exceed the largest
            // kept. A list of fewer than k - 1 others leaves the row unfinished
            // whatever its bound.
            const float lb = slast[r] * lb_scale;
            const float ub = kept_max * (1.f + dl) * (1.f + 1e-6f);
            certified = nkept == kk && lb > ub;
        } else {
            // no bound on the dropped candidates (learned routing): the row is
            // only completed by the exact scan when too few candidates were found
            certified = nvalid >= kk;
        }
    }
    if (!slast) flags |= KVB_ROW_UNCERTIFIED;
    if (force_period > 0 && (i % force_period) == 0) certified = false;
    if (!certified) {
        flags |= KVB_ROW_FALLBACK;
        if (lane == 0) {
            const int slot = atomicAdd(fb_count, 1);
            fb_list[slot] = i;
            fb_bound[slot] = bound;
        }
    }
    if (flags_out && lane == 0) flags_out[i] = flags;
}

// -------------------------------------------------------------------- fallback
// Exact float64 selection for the listed rows, ranked by (d, j).
//
// Bounded pass (rows with a finite bound B >= their true (k-1)-th distance,
// the first FB_MAX_ROWS listed): every block takes chunks of FB_CHUNK samples
// and, row after row (the chunk stays in cache), appends the samples j != i
// with d(i, j) <= B to the row's buffer of FB_CAP entries. All of the row's
// k-1 nearest are among them, so when the buffer holds between k-1 and FB_CAP
// entries the row is finished by ranking the buffer.
//
// Full scan (every other row): an 8-pass radix select on the bits of the
// float64 squared distance (non-negative doubles order like their bit
// patterns) finds the (k-1)-th smallest value V; the neighbours are all j with
// d < V plus the smallest-index j with d == V.
//
// Both compute d in the order of dist2_f64, so they agree on every value and tie.
constexpr int FB_THREADS = 256;
constexpr int FB_CHUNK = 1024;

// m <= FB_LDS_M: blocks stage FB_STAGE consecutive samples in LDS (coalesced,
// row stride m + 1 against bank conflicts), and the listed rows' coordinates,
// bounds and ids once per chunk of up to FB_ROW_FLOATS / m rows; every
// wavefront takes listed rows in turn, one staged sample per lane. A float32
// distance screens each pair first: it errs from the exact one by at most
// (m + 3) 2^-24 relative, so a pair whose float32 distance exceeds the bound by
// (m + 10) 2^-24 cannot be within it; the others are decided in float64 in the
// summation order of dist2_f64.
constexpr int FB_STAGE = 64;
constexpr int FB_LDS_M = 192;
constexpr int FB_LDS_BYTES = 60 * 1024;   // LDS per block: the sample stage, then row chunks
constexpr int FB_ROW_FLOATS = 8192;       // at most this many row coordinates per chunk

// listed rows per LDS chunk: their coordinates (m floats), bound and id each
__host__ __device__ inline int fb_rows_per_chunk(int m)
{
    const int stage = FB_STAGE * (m + 1) * 4;
    int r = (FB_LDS_BYTES - stage) / (4 * m + 12);
    r = r < FB_ROW_FLOATS / m ? r : FB_ROW_FLOATS / m;
    return r < FB_MAX_ROWS ? (r > 1 ? r : 1) : FB_MAX_ROWS;
}
size_t fb_collect_lds_bytes(int m)
{
    const int rch = fb_rows_per_chunk(m);
    return sizeof(float) * (static_cast<size_t>(FB_STAGE) * (m + 1) + static_cast<size_t>(rch) * m) +
           (sizeof(double) + sizeof(int)) * static_cast<size_t>(rch);
}

__global__ __launch_bounds__(FB_THREADS) void k_fb_collect_lds(const float* __restrict__ X, int n, int m,
                                                               const int* __restrict__ fb_count,
                                                               const int* __restrict__ fb_list,
                                                               const float* __restrict__ fb_bound, int rows_cap,
                                                               int* __restrict__ cnt, double* __restrict__ bd,
                                                               int* __restrict__ bj)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char fb_smem[];
    const int total = min(*fb_count, rows_cap);
    if (total == 0) return;
    const int rch = fb_rows_per_chunk(m);
    const int ld = m + 1;
    double* rb = reinterpret_cast<double*>(fb_smem);                  // [rch] screened bounds
    float* xc = reinterpret_cast<float*>(rb + rch);                    // [FB_STAGE][m + 1] samples
    float* xr = xc + FB_STAGE * ld;                                    // [rch][m] listed rows
    int* ri = reinterpret_cast<int*>(xr + static_cast<size_t>(rch) * m);   // [rch] their ids
    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = threadIdx.x / WAVE;
    const double slack = 1.0 + (m + 10) * 0x1p-24;
    for (int r0 = 0; r0 < total; r0 += rch) {
        const int nr = min(rch, total - r0);
        __syncthreads();
        for (int t = threadIdx.x; t < nr; t += FB_THREADS) {
            const float B = fb_bound[r0 + t];
            ri[t] = fb_list[r0 + t];
            rb[t] = B < __uint_as_float(0x7F800000u) ? static_cast<double>(B) : -1.0;   // -1: no bound
        }
        for (int e = threadIdx.x; e < nr * m; e += FB_THREADS) {
            const int t = e / m, c = e - t * m;
            xr[e] = X[static_cast<size_t>(fb_list[r0 + t]) * m + c];
        }
        for (int c0 = blockIdx.x * FB_STAGE; c0 < n; c0 += gridDim.x * FB_STAGE) {
            __syncthreads();
            for (int e = threadIdx.x; e < FB_STAGE * m; e += FB_THREADS) {
                const int r = e / m, c = e - r * m;
                xc[r * ld + c] = c0 + r < n ? X[static_cast<size_t>(c0) * m + e] : 0.f;
            }
            __syncthreads();
            const int j = c0 + lane;
            const float* xj = xc + lane * ld;
            for (int t = wave; t < nr; t += FB_THREADS / WAVE) {
                const double B = rb[t];
                if (B < 0.0) continue;
                const int i = ri[t];
                if (j >= n || j == i) continue;
                const float* xi = xr + t * m;
                float d32 = 0.f;
                for (int c = 0; c < m; ++c) {
                    const float u = xi[c] - xj[c];
                    d32 = fmaf(u, u, d32);
                }
                if (d32 < __uint_as_float(0x7F800000u) && static_cast<double>(d32) > B * slack) continue;
                double d = 0.0;
                for (int c = 0; c < m; ++c) {
                    const double u = static_cast<double>(xi[c]) - static_cast<double>(xj[c]);
                    d = fma(u, u, d);
                }
                if (d <= B) {
                    const int slot = atomicAdd(&cnt[r0 + t], 1);
                    if (slot < FB_CAP) {
                        bd[static_cast<size_t>(r0 + t) * FB_CAP + slot] = d;
                        bj[static_cast<size_t>(r0 + t) * FB_CAP + slot] = j;
                    }
                }
            }
        }
    }
}

// m <= 16: every wavefront takes its own chunks of 64 samples, one per lane,
// with the sample's coordinates in registers (read straight from X: a chunk is
// 64 m consecutive floats), and the listed rows' coordinates, padded to 16,
// as four broadcast float4 reads from LDS; the padding adds exact zeros to
// both sums. Screen and decision as in k_fb_collect_lds.
constexpr int FB_REG_M = 16;
constexpr int FB_REG_ROWS = 768;   // listed rows per LDS chunk (76 bytes each: 57 KB)

size_t fb_collect_reg_bytes() { return static_cast<size_t>(FB_REG_ROWS) * (FB_REG_M * sizeof(float) + sizeof(double) + sizeof(int)); }

__global__ __launch_bounds__(FB_THREADS) void k_fb_collect_reg(const float* __restrict__ X, int n, int m,
                                                               const int* __restrict__ fb_count,
                                                               const int* __restrict__ fb_list,
                                                               const float* __restrict__ fb_bound, int rows_cap,
                                                               int* __restrict__ cnt, double* __restrict__ bd,
                                                               int* __restrict__ bj)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char fb_smem[];
    const int total = min(*fb_count, rows_cap);
    if (total == 0) return;
    float4* xr = reinterpret_cast<float4*>(fb_smem);                                 // [FB_REG_ROWS][4]
    double* rb = reinterpret_cast<double*>(fb_smem + FB_REG_ROWS * FB_REG_M * 4);    // [FB_REG_ROWS]
    int* ri = reinterpret_cast<int*>(rb + FB_REG_ROWS);                              // [FB_REG_ROWS]
    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = threadIdx.x / WAVE;
    const double slack = 1.0 + (m + 10) * 0x1p-24;
    for (int r0 = 0; r0 < total; r0 += FB_REG_ROWS) {
        const int nr = min(FB_REG_ROWS, total - r0);
        __syncthreads();
        for (int t = threadIdx.x; t < nr; t += FB_THREADS) {
            const float B = fb_bound[r0 + t];
            ri[t] = fb_list[r0 + t];
            rb[t] = B < __uint_as_float(0x7F800000u) ? static_cast<double>(B) : -1.0;   // -1: no bound
        }
        float* xrf = reinterpret_cast<float*>(xr);
        for (int e = threadIdx.x; e < nr * FB_REG_M; e += FB_THREADS) {
            const int t = e / FB_REG_M, c = e - t * FB_REG_M;
            xrf[e] = c < m ? X[static_cast<size_t>(fb_list[r0 + t]) * m + c] : 0.f;
        }
        __syncthreads();
        for (int c0 = (blockIdx.x * (FB_THREADS / WAVE) + wave) * WAVE; c0 < n;
             c0 += gridDim.x * FB_THREADS) {
            const int j = c0 + lane;
            float xj[FB_REG_M];
#pragma unroll
            for (int c = 0; c < FB_REG_M; ++c) xj[c] = (j < n && c < m) ? X[static_cast<size_t>(j) * m + c] : 0.f;
            for (int t = 0; t < nr; ++t) {
                const double B = rb[t];
                if (B < 0.0) continue;
                float xi[FB_REG_M];
#pragma unroll
                for (int q = 0; q < FB_REG_M / 4; ++q) {
                    const float4 v = xr[t * (FB_REG_M / 4) + q];
                    xi[4 * q] = v.x;
                    xi[4 * q + 1] = v.y;
                    xi[4 * q + 2] = v.z;
                    xi[4 * q + 3] = v.w;
                }
                float d32 = 0.f;
#pragma unroll
                for (int c = 0; c < FB_REG_M; ++c) {
                    const float u = xi[c] - xj[c];
                    d32 = fmaf(u, u, d32);
                }
                const bool near = !(d32 < __uint_as_float(0x7F800000u)) || static_cast<double>(d32) <= B * slack;
                if (near && j < n && j != ri[t]) {
                    double d = 0.0;
#pragma unroll
                    for (int c = 0; c < FB_REG_M; ++c) {
                        const double u = static_cast<double>(xi[c]) - static_cast<double>(xj[c]);
                        d = fma(u, u, d);
                    }
                    if (d <= B) {
                        const int slot = atomicAdd(&cnt[r0 + t], 1);
                        if (slot < FB_CAP) {
                            bd[static_cast<size_t>(r0 + t) * FB_CAP + slot] = d;
                            bj[static_cast<size_t>(r0 + t) * FB_CAP + slot] = j;
                        }
                    }
                }
            }
        }
    }
}

__global__ __launch_bounds__(FB_THREADS) void k_fb_collect(const float* __restrict__ X, int n, int m,
                                                           const int* __restrict__ fb_count,
                                                           const int* __restrict__ fb_list,
                                                           const float* __restrict__ fb_bound, int rows_cap,
                                                           int* __restrict__ cnt, double* __restrict__ bd,
                                                           int* __restrict__ bj)
{
    __shared__ float xs[1024];
    const int total = min(*fb_count, rows_cap);
    for (int c0 = blockIdx.x * FB_CHUNK; c0 < n && total > 0; c0 += gridDim.x * FB_CHUNK) {
        for (int t = 0; t < total; ++t) {
            const float B = fb_bound[t];
            if (!(B < __uint_as_float(0x7F800000u))) continue;
            const int i = fb_list[t];
            __syncthreads();
            for (int c = threadIdx.x; c < m; c += FB_THREADS) xs[c] = X[static_cast<size_t>(i) * m + c];
            __syncthreads();
            const double Bd = static_cast<double>(B);
#pragma unroll
            for (int u = 0; u < FB_CHUNK / FB_THREADS; ++u) {
                const int j = c0 + u * FB_THREADS + threadIdx.x;
                if (j < n && j != i) {
                    const double d = dist2_f64(xs, X + static_cast<size_t>(j) * m, m);
                    if (d <= Bd) {
                        const int slot = atomicAdd(&cnt[t], 1);
                        if (slot < FB_CAP) {
                            bd[static_cast<size_t>(t) * FB_CAP + slot] = d;
                            bj[static_cast<size_t>(t) * FB_CAP + slot] = j;
                        }
                    }
                }
            }
        }
    }
}

// The row count is *fb_count, or `count` when fb_count is null. Results go to
// row i of idx_out / d2_out, or with `compact` to row t (the list position);
// in compact mode a listed id outside [0, n) yields a row of -1 / NaN.
__global__ __launch_bounds__(FB_THREADS) void k_fallback(const float* __restrict__ X, int n, int m, int k,
                                                         const int* __restrict__ fb_count, int count,
                                                         const int* __restrict__ fb_list, int compact,
                                                         int rows_cap, const int* __restrict__ cnt,
                                                         const double* __restrict__ bd, const int* __restrict__ bj,
                                                         int32_t* __restrict__ idx_out,
                                                         float* __restrict__ d2_out)
{
    __shared__ double s_bd[FB_CAP];
    __shared__ int s_bj[FB_CAP];
    __shared__ unsigned int hist[256];
    __shared__ unsigned long long s_prefix;
    __shared__ int s_remaining;
    __shared__ double cd[256];
    __shared__ int cj[256];
    __shared__ int s_cnt_lt, s_cnt_eq;
    __shared__ int wsum_lt[FB_THREADS / WAVE], wsum_eq[FB_THREADS / WAVE];
    const int tid = threadIdx.x;
    const int total = fb_count ? *fb_count : count;
    const int kk = k - 1;
    for (int t = blockIdx.x; t < total; t += gridDim.x) {
        const int i = fb_list[t];
        const size_t orow = compact ? static_cast<size_t>(t) : static_cast<size_t>(i);
        if (i < 0 || i >= n) {
            if (compact)
                for (int r = tid; r < k; r += FB_THREADS) {
                    idx_out[orow * k + r] = -1;
                    d2_out[orow * k + r] = __uint_as_float(0x7FC00000u);
                }
            continue;
        }
        const float* xi = X + static_cast<size_t>(i) * m;
        if (kk == 0) {
            if (tid == 0) {
                idx_out[orow * k] = i;
                d2_out[orow * k] = 0.f;
            }
            continue;
        }
        const int c = (cnt && t < rows_cap) ? cnt[t] : -1;
        if (c >= kk && c <= FB_CAP) {
            // bounded pass: rank the buffer by (d, j)
            for (int e = tid; e < c; e += FB_THREADS) {
                s_bd[e] = bd[static_cast<size_t>(t) * FB_CAP + e];
                s_bj[e] = bj[static_cast<size_t>(t) * FB_CAP + e];
            }
            __syncthreads();
            for (int e = tid; e < c; e += FB_THREADS) {
                const double d = s_bd[e];
                const int j = s_bj[e];
                int rank = 0;
                for (int u = 0; u < c; ++u) rank += (s_bd[u] < d) || (s_bd[u] == d && s_bj[u] < j);
                if (rank < kk) {
                    idx_out[orow * k + 1 + rank] = j;
                    d2_out[orow * k + 1 + rank] = static_cast<float>(d);
                }
            }
            if (tid == 0) {
                idx_out[orow * k] = i;
                d2_out[orow * k] = 0.f;
            }
            __syncthreads();
            continue;
        }
        if (tid == 0) {
            s_prefix = 0ull;
            s_remaining = kk;
        }
        __syncthreads();
        for (int shift = 56; shift >= 0; shift -= 8) {
            hist[tid] = 0u;
            __syncthreads();
            const unsigned long long pfx = s_prefix;
            const unsigned long long pmask = (shift == 56) ? 0ull : (~0ull << (shift + 8));
            for (int j = tid; j < n; j += FB_THREADS) {
                if (j == i) continue;
                const double d = dist2_f64(xi, X + static_cast<size_t>(j) * m, m);
                const unsigned long long u = static_cast<unsigned long long>(__double_as_longlong(d));
                if ((u & pmask) == pfx) atomicAdd(&hist[(u >> shift) & 255ull], 1u);
            }
            __syncthreads();
            if (tid == 0) {
                int rem = s_remaining;
                int b = 0;
                for (; b < 256; ++b) {
                    if (static_cast<int>(hist[b]) >= rem) break;
                    rem -= static_cast<int>(hist[b]);
                }
                s_prefix = pfx | (static_cast<unsigned long long>(b) << shift);
                s_remaining = rem;
            }
            __syncthreads();
        }
        const double V = __longlong_as_double(static_cast<long long>(s_prefix));
        const int need_eq = s_remaining;      // how many d == V entries to take
        const int n_lt = kk - need_eq;        // entries with d < V
        if (tid == 0) {
            s_cnt_lt = 0;
            s_cnt_eq = 0;
        }
        __syncthreads();
        // ordered compaction in index order
        for (int j0 = 0; j0 < n; j0 += FB_THREADS) {
            const int j = j0 + tid;
            double d = 0.0;
            bool lt = false, eq = false;
            if (j < n && j != i) {
                d = dist2_f64(xi, X + static_cast<size_t>(j) * m, m);
                lt = d < V;
                eq = d == V;
            }
            const uint64_t bl = __ballot(lt), be = __ballot(eq);
            const int w = tid / WAVE;
            if ((tid & (WAVE - 1)) == 0) {
                wsum_lt[w] = __popcll(bl);
                wsum_eq[w] = __popcll(be);
            }
            __syncthreads();
            int off_lt = s_cnt_lt, off_eq = s_cnt_eq;
            for (int u = 0; u < w; ++u) {
                off_lt += wsum_lt[u];
                off_eq += wsum_eq[u];
            }
            if (lt) {
                const int p = off_lt + mbcnt64(bl);
                cd[p] = d;
                cj[p] = j;
            }
            if (eq) {
                const int p = off_eq + mbcnt64(be);
                if (p < need_eq) {
                    cd[n_lt + p] = d;
                    cj[n_lt + p] = j;
                }
            }
            __syncthreads();
            if (tid == 0) {
                int a = 0, b = 0;
                for (int u = 0; u < FB_THREADS / WAVE; ++u) {
                    a += wsum_lt[u];
                    b += wsum_eq[u];
                }
                s_cnt_lt += a;
                s_cnt_eq += b;
            }
            __syncthreads();
        }
        // rank by (d, j) and write
        if (tid < kk) {
            const double d = cd[tid];
            const int j = cj[tid];
            int rank = 0;
            for (int u = 0; u < kk; ++u) rank += (cd[u] < d) || (cd[u] == d && cj[u] < j);
            idx_out[orow * k + 1 + rank] = j;
            d2_out[orow * k + 1 + rank] = static_cast<float>(d);
        }
        if (tid == 0) {
            idx_out[orow * k] = i;
            d2_out[orow * k] = 0.f;
        }
        __syncthreads();
    }
}

// -------------------------------------------------------------------- launchers
int spatial_bbox_blocks(int n) { return std::max(1, std::min(1024, (n + 4095) / 4096)); }
int spatial_tiles(int n) { return (n + TILE - 1) / TILE; }
int spatial_superblocks(int n) { return (spatial_tiles(n) + SB_TILES - 1) / SB_TILES; }

// Bits per coordinate of the Morton code: enough cells for a few samples each
// (the tiles stay compact; finer codes only lengthen the sort), at most 32 in all.
int spatial_code_bits(int n, int m)
{
    int lg = 0;
    while ((1ll << lg) < static_cast<long long>(n)) ++lg;
    const int want = std::max(8, (lg + m - 1) / m + 2);
    return std::min(std::min(31, 32 / m), want);
}

hipError_t launch_spatial_codes(const float* X, int n, int m, float* bbox_part, uint32_t* code, int32_t* vals,
                                hipStream_t st)
{
    if (m < 1 || m > 8) return hipErrorInvalidValue;
    const int bits = spatial_code_bits(n, m);
    const int nb = spatial_bbox_blocks(n);
    const int rpb = (n + nb - 1) / nb;
    auto boxes = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nb), dim3(BBOX_THREADS), 0, st, X, n, rpb, bbox_part);
    };
    switch (m) {
    case 1: boxes(k_bbox_partial<1>); break;
    case 2: boxes(k_bbox_partial<2>); break;
    case 3: boxes(k_bbox_partial<3>); break;
    case 4: boxes(k_bbox_partial<4>); break;
    case 5: boxes(k_bbox_partial<5>); break;
    case 6: boxes(k_bbox_partial<6>); break;
    case 7: boxes(k_bbox_partial<7>); break;
    default: boxes(k_bbox_partial<8>); break;
    }
    hipLaunchKernelGGL(k_morton, dim3((n + 255) / 256), dim3(256), 0, st, X, n, m, bits, bbox_part, nb, code, vals);
    return hipGetLastError();
}

hipError_t launch_spatial_layout(const float* X, int n, int m, const int32_t* perm, float* Xs, float* tbox,
                                 float* sbox, hipStream_t st)
{
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(spatial_superblocks(n)), dim3(LAYOUT_THREADS), 0, st, X, n, perm, Xs, tbox,
                           sbox);
        return hipGetLastError();
    };
    switch (m) {
    case 1: return go(k_spatial_layout<1>);
    case 2: return go(k_spatial_layout<2>);
    case 3: return go(k_spatial_layout<3>);
    case 4: return go(k_spatial_layout<4>);
    case 5: return go(k_spatial_layout<5>);
    case 6: return go(k_spatial_layout<6>);
    case 7: return go(k_spatial_layout<7>);
    case 8: return go(k_spatial_layout<8>);
    default: return hipErrorInvalidValue;
    }
}

template <int M, int R>
static hipError_t launch_select_r(const SpatialView& sv, int n, int kp, uint64_t* keys, float* slast,
                                  unsigned long long* pairs, hipStream_t st)
{
    const int rows_per_block = 4 * R;
    const dim3 grid((n + rows_per_block - 1) / rows_per_block), block(256);
    if (kp <= 64)
        hipLaunchKernelGGL((k_select_direct<M, R, 1>), grid, block, 0, st, sv, n, kp, keys, slast, pairs);
    else if (kp <= 128)
        hipLaunchKernelGGL((k_select_direct<M, R, 2>), grid, block, 0, st, sv, n, kp, keys, slast, pairs);
    else
        hipLaunchKernelGGL((k_select_direct<M, R, 4>), grid, block, 0, st, sv, n, kp, keys, slast, pairs);
    return hipGetLastError();
}

// Rows per wavefront: more rows share a tile's loads and box tests, but scan each
// other's tiles. Up to five coordinates one while the rows are few enough for every
// wavefront to be resident at once (sphere, n = 2000: 14 us at 1 row, 21 at 2, 28 at
// 3; 32000: 142 against 143), two beyond (torus, n = 100k: 183 us at 1, 170 at 2, 180
// at 3; 1M: 3.19, 2.82 and 2.80 ms). From six on a row's tiles are many and mostly its
// neighbours' too: two (n = 30k, m = 8, k = 64: 0.72 ms at 1, 0.62 at 2), and three for lists
// of up to 128 of many samples (n = 300k, k = 16: 17.5 ms at 2, 16.4 at 3; longer lists fill
// the LDS: k = 160 28.1 and 29.3).
constexpr int SELECT_ONE_ROW = 32768, SELECT_THREE_ROWS = 262144;

template <int M>
static hipError_t launch_select_m(const SpatialView& sv, int n, int kp, uint64_t* keys, float* slast,
                                  unsigned long long* pairs, hipStream_t st)
{
    if constexpr (M >= 6) {
        if (n > SELECT_THREE_ROWS && kp <= 128) return launch_select_r<M, 3>(sv, n, kp, keys, slast, pairs, st);
    } else {
        if (n <= SELECT_ONE_ROW) return launch_select_r<M, 1>(sv, n, kp, keys, slast, pairs, st);
    }
    return launch_select_r<M, 2>(sv, n, kp, keys, slast, pairs, st);
}

hipError_t launch_select_direct(const float* Xs, const float* tbox, const float* sbox, int n, int m, int kp,
                                uint64_t* keys, float* slast, unsigned long long* pairs, hipStream_t st)
{
    const SpatialView sv = {Xs, tbox, sbox};
    switch (m) {
    case 1: return launch_select_m<1>(sv, n, kp, keys, slast, pairs, st);
    case 2: return launch_select_m<2>(sv, n, kp, keys, slast, pairs, st);
    case 3: return launch_select_m<3>(sv, n, kp, keys, slast, pairs, st);
    case 4: return launch_select_m<4>(sv, n, kp, keys, slast, pairs, st);
    case 5: return launch_select_m<5>(sv, n, kp, keys, slast, pairs, st);
    case 6: return launch_select_m<6>(sv, n, kp, keys, slast, pairs, st);
    case 7: return launch_select_m<7>(sv, n, kp, keys, slast, pairs, st);
    case 8: return launch_select_m<8>(sv, n, kp, keys, slast, pairs, st);
    default: return hipErrorInvalidValue;
    }
}

template <int LPC, bool CV>
static void launch_refine_l(const float* X, int n, int m, int k, int kp, int kstride, const uint64_t* keys,
                            const float* slast, float lb_scale, int32_t* idx, float* d2, int32_t* flags, int* fb_count,
                            int* fb_list, float* fb_bound, int force_period, const float* Xs, const int32_t* perm,
                            const int32_t* order, hipStream_t st)
{
    const dim3 grid((n + 3) / 4), block(256);
    if (kp <= 64)
        hipLaunchKernelGGL((k_refine<1, LPC, CV>), grid, block, 0, st, X, n, m, k, kp, kstride, keys, slast, lb_scale,
                           idx, d2, flags, fb_count, fb_list, fb_bound, force_period, Xs, perm, order);
    else if (kp <= 128)
        hipLaunchKernelGGL((k_refine<2, LPC, CV>), grid, block, 0, st, X, n, m, k, kp, kstride, keys, slast, lb_scale,
                           idx, d2, flags, fb_count, fb_list, fb_bound, force_period, Xs, perm, order);
    else
        hipLaunchKernelGGL((k_refine<4, LPC, CV>), grid, block, 0, st, X, n, m, k, kp, kstride, keys, slast, lb_scale,
                           idx, d2, flags, fb_count, fb_list, fb_bound, force_period, Xs, perm, order);
}

hipError_t launch_refine(const float* X, int n, int m, int k, int kp, int kstride, const uint64_t* keys,
                         const float* slast, float lb_scale, int32_t* idx, float* d2, int32_t* flags,
                         int* fb_count, int* fb_list, float* fb_bound, int force_period, const float* Xs,
                         const int32_t* perm, const int32_t* order, hipStream_t st)
{
    // rows of up to 24 floats stay with one lane per candidate; longer rows are
    // read by groups of lanes, each lane covering up to 4 float4 pieces (the
    // fewest lanes per candidate: more candidates per pass, fewer passes and
    // shorter group reductions)
#define KVB_REFINE(LPC)                                                                                              \
    do {                                                                                                              \
        if (perm)                                                                                                     \
            launch_refine_l<LPC, true>(X, n, m, k, kp, kstride, keys, slast, lb_scale, idx, d2, flags, fb_count,     \
                                       fb_list, fb_bound, force_period, Xs, perm, nullptr, st);                                \
        else                                                                                                          \
            launch_refine_l<LPC, false>(X, n, m, k, kp, kstride, keys, slast, lb_scale, idx, d2, flags, fb_count,    \
                                        fb_list, fb_bound, force_period, nullptr, nullptr, order, st);                       \
    } while (0)
    if (m <= 24)
        KVB_REFINE(0);
    else if (m <= 64)
        KVB_REFINE(4);
    else if (m <= 128)
        KVB_REFINE(8);
    else if (m <= 256)
        KVB_REFINE(16);
    else if (m <= 1024)
        KVB_REFINE(64);
    else
        return hipErrorInvalidValue;
#undef KVB_REFINE
    return hipGetLastError();
}

hipError_t launch_gather_rows(const float* X, int n, int m, const int32_t* perm, float* Xs, hipStream_t st)
{
    gather_rows(X, n, m, perm, Xs, st);
    return hipGetLastError();
}

int fallback_rows_cap(int n) { return n < FB_MAX_ROWS ? n : FB_MAX_ROWS; }

hipError_t launch_fallback(const float* X, int n, int m, int k, const int* fb_count, const int* fb_list,
                           const FallbackWork& fw, int32_t* idx, float* d2, hipStream_t st)
{
    if (m > 1024) return hipErrorInvalidValue;
    const int cap = fallback_rows_cap(n);
    hipError_t e = hipMemsetAsync(fw.cnt, 0, static_cast<size_t>(cap) * sizeof(int), st);
    if (e != hipSuccess) return e;
    if (m <= FB_REG_M) {
        const int waves = (n + WAVE - 1) / WAVE, blocks = (waves + FB_THREADS / WAVE - 1) / (FB_THREADS / WAVE);
        hipLaunchKernelGGL(k_fb_collect_reg, dim3(blocks < 2048 ? blocks : 2048), dim3(FB_THREADS),
                           fb_collect_reg_bytes(), st, X, n, m, fb_count, fb_list, fw.bound, cap, fw.cnt, fw.bd,
                           fw.bj);
    } else if (m <= FB_LDS_M) {
        const int stages = (n + FB_STAGE - 1) / FB_STAGE;
        hipLaunchKernelGGL(k_fb_collect_lds, dim3(stages < 2048 ? stages : 2048), dim3(FB_THREADS),
                           fb_collect_lds_bytes(m), st, X, n, m, fb_count, fb_list, fw.bound, cap, fw.cnt, fw.bd,
                           fw.bj);
    } else {
        const int chunks = (n + FB_CHUNK - 1) / FB_CHUNK;
        hipLaunchKernelGGL(k_fb_collect, dim3(chunks < 2048 ? chunks : 2048), dim3(FB_THREADS), 0, st, X, n, m,
                           fb_count, fb_list, fw.bound, cap, fw.cnt, fw.bd, fw.bj);
    }
    hipLaunchKernelGGL(k_fallback, dim3(512), dim3(FB_THREADS), 0, st, X, n, m, k, fb_count, 0, fb_list, 0, cap,
                       fw.cnt, fw.bd, fw.bj, idx, d2);
    return hipGetLastError();
}

hipError_t launch_exact_rows(const float* X, int n, int m, int k, const int* rows, int nrows, int32_t* idx, float* d2,
                             hipStream_t st)
{
    if (nrows <= 0) return hipSuccess;
    const int grid = nrows < 1024 ? nrows : 1024;
    hipLaunchKernelGGL(k_fallback, dim3(grid), dim3(FB_THREADS), 0, st, X, n, m, k, nullptr, nrows, rows, 1, 0,
                       nullptr, nullptr, nullptr, idx, d2);
    return hipGetLastError();
}

}  // namespace kvb
