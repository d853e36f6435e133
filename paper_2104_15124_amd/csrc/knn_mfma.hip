// Matrix-core distance tiles for the k-NN selection (gfx950 MFMA).
//
// For m >= 9 the squared distances are a dense contraction: with samples
// centred on their column mean (y = x - mu), the selection score
//   s_ij = |y_j|^2 - 2 y_i . y_j = |y_i - y_j|^2 - |y_i|^2
// ranks the candidates j of row i exactly like the squared distance. It is one
// GEMM-shaped product of a query operand and a candidate operand, both laid
// out by the prep kernel with the norm folded into the contraction:
//   query     a_i = [-2 t_1(y_i), ..., -2 t_P(y_i), 1, 1, 1, 0...]
//   candidate b_j = [  u_1(y_j), ...,    u_P(y_j), n1, n2, n3, 0...]
// so that a_i . b_j = s_ij up to the rounding of the operands. In BF16 mode the
// coordinates are split into two or three BF16 terms (hi + lo, or
// hi + mid + lo) and the product pairs listed below; the norm is split into
// three BF16 terms. In FP32 mode the operands are y itself.
//
// Tiles are 32 queries x 32 candidates (v_mfma_f32_32x32x16_bf16 or
// v_mfma_f32_32x32x2_f32, FP32 accumulation). A workgroup of four or eight
// wavefronts stages 32 candidates at a time in LDS (two stages; the next tile
// is prefetched into registers while the current one is consumed); every
// wavefront keeps its query fragments in registers and loads a stage's
// candidate fragments in one batch before the MFMA chain. Scores at or below a query's threshold are appended
// to that query's LDS buffer; a buffer that may not absorb another tile is merged into
// the query's sorted list (in global scratch) by the wavefront bitonic merge,
// which lowers the threshold.
//
// Certificate bound. After the scan, every candidate that is not on a row's
// list has a score >= s_last (the list's last score). The epilogue turns
// s_last into a lower bound on the true squared distance of any such
// candidate, from the operand and accumulation error model:
//   |x_i - x_j|^2 >= (sqrt(max(0, s_last + |y_i|^2 - E_i)) - c (|y_i| + R))^2,
//   E_i = g (R + 1.05 |y_i|)^2 + h R^2 + x |y_i| R,
// with R = max_j |y_j|, g the accumulation bound (K + 4) 2^-24, h the norm
// representation bound, x the cross-term bound of the chosen split and c the
// centring rounding bound. The refine step compares it with the largest kept
// exact distance.
#include "knn_mfma_common.h"

namespace kvb {

// ------------------------------------------------------------------ prep
// Column sums (float64) over blocks of rows, then the fixed-order mean. For
// m <= 256 the block's threads form T = 256 / m row lanes of m columns: thread
// (j, c) sums column c over rows r0 + j, r0 + j + T, ... (consecutive threads
// read consecutive columns of a row), and the T partial sums of a column are
// added in the order j = 0, 1, ... . Wider rows: one thread per column. Bound
// by the chain of loads of a block's rows: eight are in flight, and a block
// takes 128 rows up to 1024 blocks (4096 rows per block left 8 blocks at n =
// 30k, 1.0 ms for m = 200, 0.02 now; 0.97 -> 0.38 ms at n = 4M, m = 128).
__global__ __launch_bounds__(256) void k_colsum_partial(const float* __restrict__ X, int n, int m, int rows_per_block,
                                                        double* __restrict__ part)
{
    __shared__ double s_part[256];
    const int r0 = blockIdx.x * rows_per_block;
    const int r1 = min(n, r0 + rows_per_block);
    if (m <= 256) {
        const int T = 256 / m;
        const int j = threadIdx.x / m, c = threadIdx.x % m;
        double s = 0.0;
        if (j < T) {
#pragma unroll 8
            for (int r = r0 + j; r < r1; r += T) s += static_cast<double>(X[static_cast<size_t>(r) * m + c]);
        }
        s_part[threadIdx.x] = s;
        __syncthreads();
        if (threadIdx.x < m) {
            double t = 0.0;
            for (int q = 0; q < T; ++q) t += s_part[q * m + threadIdx.x];
            part[static_cast<size_t>(blockIdx.x) * m + threadIdx.x] = t;
        }
        return;
    }
    for (int c = threadIdx.x; c < m; c += blockDim.x) {
        double s = 0.0;
#pragma unroll 8
        for (int r = r0; r < r1; ++r) s += static_cast<double>(X[static_cast<size_t>(r) * m + c]);
        part[static_cast<size_t>(blockIdx.x) * m + c] = s;
    }
}

// The block partials of each column added in a fixed order, one wavefront per column.
__global__ __launch_bounds__(WAVE) void k_colsum_finish(const double* __restrict__ part, int nb, int m, int n,
                                                        double* __restrict__ mu)
{
    const int c = blockIdx.x;
    double s = 0.0;
#pragma unroll 4
    for (int b = threadIdx.x; b < nb; b += WAVE) s += part[static_cast<size_t>(b) * m + c];
    s = wave_sum_f64(s);
    if (threadIdx.x == 0) mu[c] = s / static_cast<double>(n);
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f)
{
    const uint32_t u = __float_as_uint(f);
    const uint32_t r = ((u >> 16) & 1u) + 0x7FFFu;
    return static_cast<uint16_t>((u + r) >> 16);
}
__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float(static_cast<uint32_t>(h) << 16); }

// Position of candidate-operand element (row i, column c) in the tile-major
// fragment order used by the selection kernel: 32-row tiles, each laid out as
// [k-step][lane half][row][fragment element], i.e. exactly the LDS image that
// the MFMA B-operand reads, so a tile streams in with contiguous copies.
__device__ __forceinline__ size_t bpos(int i, int c, int kpad, int kstep, int vec)
{
    const int s = c / kstep, w = c % kstep, h = w / vec, v = w % vec;
    return static_cast<size_t>(i / 32) * 32 * kpad + ((s * 2 + h) * 32 + (i % 32)) * vec + v;
}

// One wavefront per row: y = x - mu (float32), the operand terms, |y|^2
// (float64, kept as float32 for the certificate) and the running max |y|.
// split: 0 = float32 operands, 1 = one BF16 term, 3 = hi/lo pairs, 6 = hi/mid/lo pairs.
// Rows n..npad-1 pad the last 32-row tile with zeros. With brow non-null the
// candidate operand row of sample i is written at row brow[i] instead of i
// (the bucket order of the learned partitioner; npad == n).
// sum over aligned groups of lpr lanes (16, 32 or 64), every lane of a group
// receiving it; the xor stages below lpr are those of wave_sum_f64, so where
// the lanes of a group beyond the row hold 0 the row's sum is the same
__device__ __forceinline__ double group_sum_f64(double v, int lpr)
{
    if (lpr > 32) v += shfl_xor_f64(v, 32);
    if (lpr > 16) v += shfl_xor_f64(v, 16);
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) v += shfl_xor_f64(v, o);
    return v;
}

static int prep_blocks(int npad) { return std::max(1, std::min(4096, (npad + 3) / 4)); }

__global__ __launch_bounds__(256) void k_prep_rows(const float* __restrict__ X, int n, int npad, int m,
                                                   const double* __restrict__ mu, int split, int kpad,
                                                   void* __restrict__ Aq, void* __restrict__ Bc,
                                                   float* __restrict__ ynorm2, unsigned* __restrict__ rmax_bits,
                                                   const int* __restrict__ brow, const int* __restrict__ arow)
{
    // rows are taken in a grid-stride loop, 64 / lpr rows per wavefront (lpr
    // lanes per row, the power of two >= m from 16 on); the largest norm is
    // folded per block and published with one atomic (an atomic per row
    // serialises millions of updates of one address)
    const int lane = lane_id();
    const int lpr = m <= 16 ? 16 : m <= 32 ? 32 : WAVE;
    const int rpw = WAVE / lpr, gl = lane % lpr;
    float wmax = 0.f;
    for (int i0 = (blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * rpw; i0 < npad;
         i0 += gridDim.x * 4 * rpw) {
        const int i = i0 + lane / lpr;
        const bool live = i < npad;   // rows past npad (last wavefront): nothing written
        const bool real = i < n;
        const int ib = (brow && real) ? brow[i] : i;   // candidate operand row
        const int ia = (arow && real) ? arow[i] : i;   // query operand row
        const float* x = X + static_cast<size_t>(real ? i : 0) * m;
        double nrm = 0.0;
        if (split == 0) {
            constexpr int KS = 2, VE = 1;
            float* A = static_cast<float*>(Aq) + static_cast<size_t>(ia) * kpad;
            float* B = static_cast<float*>(Bc);
            for (int c = gl; c < m; c += lpr) {
                const float y = real ? static_cast<float>(static_cast<double>(x[c]) - mu[c]) : 0.0f;
                nrm += static_cast<double>(y) * static_cast<double>(y);
                if (real) A[c] = -2.0f * y;
                if (live) B[bpos(ib, c, kpad, KS, VE)] = y;
            }
            nrm = group_sum_f64(nrm, lpr);
            for (int c = m + gl; c < kpad; c += lpr) {
                if (real) A[c] = (c == m) ? 1.0f : 0.0f;
                if (live) B[bpos(ib, c, kpad, KS, VE)] = (c == m) ? static_cast<float>(nrm) : 0.0f;
            }
        } else {
            constexpr int KS = 16, VE = 8;
            uint16_t* A = static_cast<uint16_t*>(Aq) + static_cast<size_t>(ia) * kpad;
            uint16_t* B = static_cast<uint16_t*>(Bc);
            for (int c = gl; c < m; c += lpr) {
                const float y = real ? static_cast<float>(static_cast<double>(x[c]) - mu[c]) : 0.0f;
                nrm += static_cast<double>(y) * static_cast<double>(y);
                const uint16_t hi = f32_to_bf16_rne(y);
                const float r1 = y - bf16_to_f32(hi);
                const uint16_t mid = f32_to_bf16_rne(r1);
                const float r2 = r1 - bf16_to_f32(mid);
                const uint16_t lo = f32_to_bf16_rne(r2);
                // -2 t is exact in BF16 (a power-of-two scaling)
                const uint16_t hi2 = f32_to_bf16_rne(-2.0f * bf16_to_f32(hi));
                const uint16_t mid2 = f32_to_bf16_rne(-2.0f * bf16_to_f32(mid));
                const uint16_t lo2 = f32_to_bf16_rne(-2.0f * bf16_to_f32(lo));
                uint16_t a[6], b[6];
                int P = 1;
                if (split == 1) {
                    a[0] = hi2; b[0] = hi;
                } else if (split == 3) {                     // (hi,hi) (hi,lo) (lo,hi), the second term as lo
                    a[0] = hi2; b[0] = hi;
                    a[1] = hi2; b[1] = mid;
                    a[2] = mid2; b[2] = hi;
                    P = 3;
                } else {                                     // (hi,hi) (hi,mid) (mid,hi) (hi,lo) (lo,hi) (mid,mid)
                    a[0] = hi2; b[0] = hi;
                    a[1] = hi2; b[1] = mid;
                    a[2] = mid2; b[2] = hi;
                    a[3] = hi2; b[3] = lo;
                    a[4] = lo2; b[4] = hi;
                    a[5] = mid2; b[5] = mid;
                    P = 6;
                }
                for (int t = 0; t < P; ++t) {
                    if (real) A[t * m + c] = a[t];
                    if (live) B[bpos(ib, t * m + c, kpad, KS, VE)] = b[t];
                }
            }
            nrm = group_sum_f64(nrm, lpr);
            const int P = split;
            const uint16_t n1 = f32_to_bf16_rne(static_cast<float>(nrm));
            const double r1 = nrm - static_cast<double>(bf16_to_f32(n1));
            const uint16_t n2 = f32_to_bf16_rne(static_cast<float>(r1));
            const double r2 = r1 - static_cast<double>(bf16_to_f32(n2));
            const uint16_t n3 = f32_to_bf16_rne(static_cast<float>(r2));
            const uint16_t one = f32_to_bf16_rne(1.0f);
            for (int c = P * m + gl; c < kpad; c += lpr) {
                const int t = c - P * m;
                if (real) A[c] = t < 3 ? one : static_cast<uint16_t>(0);
                if (live)
                    B[bpos(ib, c, kpad, KS, VE)] = t == 0   ? n1
                                                   : t == 1 ? n2
                                                   : t == 2 ? n3
                                                            : static_cast<uint16_t>(0);
            }
        }
        if (real && gl == 0) {
            ynorm2[ia] = static_cast<float>(nrm);   // by query operand row
            wmax = fmaxf(wmax, static_cast<float>(sqrt(nrm) * (1.0 + 1e-6)));
        }
    }
    __shared__ float s_wmax[4];
    wmax = wave_max_f32(wmax);
    if (lane == 0) s_wmax[threadIdx.x >> 6] = wmax;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float bm = fmaxf(fmaxf(s_wmax[0], s_wmax[1]), fmaxf(s_wmax[2], s_wmax[3]));
        if (bm > 0.f) atomicMax(rmax_bits, __float_as_uint(bm));
    }
}

// k_prep_rows for FP32 operands of rows of at most PREP_THREAD_M coordinates,
// by operand row (the BF16 split terms stay with the wavefront per row, whose
// 2-byte query operand writes coalesce):
// thread r prepares operand row r from input row r (r >= n: a padding row of
// zeros), with the same values as
// k_prep_rows (|y|^2 summed over the row in column order). Consecutive
// threads then write consecutive query operand rows and, in the candidate
// operand, whose k-step blocks hold 32 consecutive rows, consecutive
// addresses.
constexpr int PREP_THREAD_M = 64;

__global__ __launch_bounds__(256) void k_prep_rows_thread(const float* __restrict__ X, int n, int npad, int m,
                                                          const double* __restrict__ mu, int split, int kpad,
                                                          void* __restrict__ Aq, void* __restrict__ Bc,
                                                          float* __restrict__ ynorm2, unsigned* __restrict__ rmax_bits)
{
    const int r = blockIdx.x * 256 + threadIdx.x;
    float wmax = 0.f;
    if (r < npad) {
        const int i = r < n ? r : -1;
        const bool real = i >= 0;
        const int ib = r, ia = r;
        const float* x = X + static_cast<size_t>(real ? i : 0) * m;
        double nrm = 0.0;
        {
            constexpr int KS = 2, VE = 1;
            float* A = static_cast<float*>(Aq) + static_cast<size_t>(ia) * kpad;
            float* B = static_cast<float*>(Bc);
            const bool vec = (m % 4 == 0) && (kpad % 4 == 0) && ((reinterpret_cast<uintptr_t>(X) & 15) == 0) &&
                             ((reinterpret_cast<uintptr_t>(Aq) & 15) == 0);
            if (vec) {
                for (int c = 0; c < m; c += 4) {
                    const float4 xv = real ? *reinterpret_cast<const float4*>(x + c) : make_float4(0.f, 0.f, 0.f, 0.f);
                    const float xs[4] = {xv.x, xv.y, xv.z, xv.w};
                    float ys[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        ys[u] = real ? static_cast<float>(static_cast<double>(xs[u]) - mu[c + u]) : 0.0f;
                        nrm += static_cast<double>(ys[u]) * static_cast<double>(ys[u]);
                        B[bpos(ib, c + u, kpad, KS, VE)] = ys[u];
                    }
                    if (real)
                        *reinterpret_cast<float4*>(A + c) = make_float4(-2.0f * ys[0], -2.0f * ys[1], -2.0f * ys[2],
                                                                        -2.0f * ys[3]);
                }
                for (int c = m; c < kpad; c += 4) {
                    float av[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        av[u] = (c + u == m) ? 1.0f : 0.0f;
                        B[bpos(ib, c + u, kpad, KS, VE)] = (c + u == m) ? static_cast<float>(nrm) : 0.0f;
                    }
                    if (real) *reinterpret_cast<float4*>(A + c) = make_float4(av[0], av[1], av[2], av[3]);
                }
            } else {
                for (int c = 0; c < m; ++c) {
                    const float y = real ? static_cast<float>(static_cast<double>(x[c]) - mu[c]) : 0.0f;
                    nrm += static_cast<double>(y) * static_cast<double>(y);
                    if (real) A[c] = -2.0f * y;
                    B[bpos(ib, c, kpad, KS, VE)] = y;
                }
                for (int c = m; c < kpad; ++c) {
                    if (real) A[c] = (c == m) ? 1.0f : 0.0f;
                    B[bpos(ib, c, kpad, KS, VE)] = (c == m) ? static_cast<float>(nrm) : 0.0f;
                }
            }
        }
        if (real) {
            ynorm2[ia] = static_cast<float>(nrm);
            wmax = static_cast<float>(sqrt(nrm) * (1.0 + 1e-6));
        }
    }
    // the block's largest norm published with one atomic (one per wavefront
    // made 125k updates of one address at n = 8M)
    __shared__ float s_wmax[4];
    wmax = wave_max_f32(wmax);
    if (lane_id() == 0) s_wmax[threadIdx.x >> 6] = wmax;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float bm = fmaxf(fmaxf(s_wmax[0], s_wmax[1]), fmaxf(s_wmax[2], s_wmax[3]));
        if (bm > 0.f) atomicMax(rmax_bits, __float_as_uint(bm));
    }
}

// ------------------------------------------------------------------ select
// WV wavefronts per workgroup share every candidate stage; each wavefront owns
// 32 queries. The first CAP / 32 tiles of a scan that starts from empty
// lists are written into the lists directly and sorted once; afterwards keys
// at or below a query's threshold collect in its LDS buffer of BUF keys, which
// is merged into the list whenever the next tile's keys would not fit.
//
// MODE 0: queries and candidates in sample order, every tile scanned.
//
// MODE 1 (learned): bucketed search of the learned partitioner. Workgroup w
// takes work item (bucket b, first query entry t0): its queries are entries
// t0 .. min(t0 + 32 WV, qptr[b + 1]) - 1 of qids, its candidates the tiles
// tptr[b] .. tptr[b + 1] - 1 of the bucket-ordered candidate operand, whose
// rows map to sample ids through cid (-1 for padding). Lists of queries are
// created on the first probe pass and merged into on later ones (the list's
// kp-th score is the starting threshold); no certificate is computed.
//
// MODE 2 (curve order): the query tiles that the tree walk handed over
// (crv.wide), a wavefront each, every tile scanned. lb_out holds their queries'
// thresholds, which the lists start from.
template <class Tr, int KS, int WV, int E, int MODE>
__global__ __launch_bounds__(64 * WV) void k_select_mfma(
    const typename Tr::elem* __restrict__ Aq,
                                                          const typename Tr::elem* __restrict__ Bc, int n, int kp,
                                                          const float* __restrict__ ynorm2,
                                                          const unsigned* __restrict__ rmax_bits, ErrModel em,
                                                          uint64_t* __restrict__ lists, float* __restrict__ lb_out,
                                                          BucketArgs ba, const int* __restrict__ wide_count,
                                                          const int* __restrict__ wide,
                                                          unsigned long long* __restrict__ pair_count)
{
    constexpr bool LEARNED = MODE == 1;
    using elem = typename Tr::elem;
    using frag = typename Tr::frag;
    constexpr int CAP = WAVE * E;
    constexpr int kpad = KS * Tr::KSTEP;        // padded contraction length
    constexpr int NQ = 32;                      // queries per wavefront
    constexpr int BUF = WV == 8 ? 48 : 64;   // per-query LDS buffer entries
    // two candidate stages, fragment-major: [stage][k-step][half][row] so that
    // lane l reads consecutive fragments (no bank conflicts). The next tile is
    // prefetched into registers while the current one is consumed.
    constexpr int STAGE_BYTES = KS * 64 * static_cast<int>(sizeof(frag));
    constexpr int CHUNKS = STAGE_BYTES / 16;                 // 16-byte pieces per tile
    constexpr int PF = (CHUNKS + 64 * WV - 1) / (64 * WV);  // pieces per thread
    __shared__ __attribute__((aligned(16))) frag s_tile[2][KS][2][32];
    __shared__ uint64_t s_buf[WV][NQ][BUF];

    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = lane >> 5;
    __shared__ int s_qid[WV][NQ];

    // query ids of this wavefront (-1: none) and the candidate tile range
    int q0 = 0, tbeg = 0, tend = 0;
    if constexpr (LEARNED) {
        const int nw = *ba.n_work;
        if (static_cast<int>(blockIdx.x) >= nw) return;   // whole workgroup
        const int2 wk = ba.work[xcd_index(blockIdx.x, nw)];   // a bucket's items on one XCD
        const int qend = ba.qptr[wk.x + 1];
        q0 = wk.y + wave * NQ;
        tbeg = ba.tptr[wk.x];
        tend = ba.tptr[wk.x + 1];
        if (lane < NQ) s_qid[wave][lane] = q0 + lane < qend ? ba.qids[q0 + lane] : -1;
    } else if constexpr (MODE == 2) {
        const int w = blockIdx.x * WV, count = *wide_count;
        if (w >= count) return;   // whole workgroup
        tend = (n + 31) / 32;
        q0 = w + wave < count ? wide[w + wave] * NQ : n;
        if (lane < NQ) s_qid[wave][lane] = q0 + lane < n ? q0 + lane : -1;
    } else {
        q0 = (blockIdx.x * WV + wave) * NQ;
        tend = (n + 31) / 32;
        if (lane < NQ) s_qid[wave][lane] = q0 + lane < n ? q0 + lane : -1;
    }
    wave_lds_sync();

    frag qa[KS];
    {
        int row = s_qid[wave][lane & 31];   // query operand row: the sample id
        if (row < 0) row = max(s_qid[wave][0], 0);
        const elem* src = Aq + static_cast<size_t>(row) * kpad + half * Tr::VEC;
#pragma unroll
        for (int s = 0; s < KS; ++s) qa[s] = Tr::load(src + s * Tr::KSTEP);
    }
    float tauv[16];
    if (LEARNED && !ba.first) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int qid = s_qid[wave][acc_row(r, half)];
            tauv[r] = qid >= 0 ? key_dist(lists[static_cast<size_t>(qid) * CAP + (kp - 1)]) : -__uint_as_float(0x7F800000u);
        }
    } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int qid = s_qid[wave][acc_row(r, half)];
            tauv[r] = MODE != 0 && qid < 0 ? -__uint_as_float(0x7F800000u)
                      : MODE == 2          ? lb_out[qid]
                                           : __uint_as_float(0x7F800000u);
        }
        for (int q = 0; q < NQ; ++q) {
            const int qg = s_qid[wave][q];
            if (qg >= 0)
                for (int t = lane; t < CAP; t += WAVE) lists[static_cast<size_t>(qg) * CAP + t] = KEY_INF;
        }
    }
    wave_lds_sync();
    const int nq_valid = __popcll(__ballot(lane < NQ && s_qid[wave][lane] >= 0));
    unsigned long long pairs = 0;

    // a tile of the tile-major candidate operand is one contiguous block, laid
    // out exactly like an LDS stage: it moves as 16-byte pieces
    // the query fragments have landed before the loop, so the only vector
    // loads in flight inside it are the next tile's prefetch
    int qrow[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) qrow[r] = s_qid[wave][acc_row(r, half)];

    __builtin_amdgcn_s_waitcnt(0);
    u32x4 pf[PF];
    int cid_pf = -1;
    int tile = tbeg < tend ? tbeg : -1;
    if (tile >= 0) {
        const u32x4* g = reinterpret_cast<const u32x4*>(Bc + static_cast<size_t>(tile) * 32 * kpad);
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int ch = threadIdx.x + u * 64 * WV;
            if (ch < CHUNKS) pf[u] = g[ch];
        }
        if constexpr (LEARNED) cid_pf = ba.cid[static_cast<size_t>(tile) * 32 + (lane & 31)];
    }
    // the buffers' fill, wave-uniform: query q's count in byte q % 4 of
    // cntw[q / 4] (every index below is a compile-time constant, so they stay
    // in scalar registers; BUF <= 64 fits a byte)
    static_assert(BUF <= 255, "a buffer count must fit a byte");
    uint32_t cntw[NQ / 4];
#pragma unroll
    for (int i = 0; i < NQ / 4; ++i) cntw[i] = 0u;
    auto cnt_of = [&](int q) { return static_cast<int>((cntw[q >> 2] >> (8 * (q & 3))) & 0xFFu); };
    // lists that start empty are filled by the first tiles without merging
    bool filling = MODE == 0 || (LEARNED && ba.first);
    const int fill_tiles = CAP / 32;   // the whole list capacity: a tighter first threshold
    for (int it = 0; tile >= 0; ++it) {
        const int stage = it & 1;
        {
            u32x4* d = reinterpret_cast<u32x4*>(&s_tile[stage][0][0][0]);
#pragma unroll
            for (int u = 0; u < PF; ++u) {
                const int ch = threadIdx.x + u * 64 * WV;
                if (ch < CHUNKS) d[ch] = pf[u];
            }
        }
        const int cid_cur = cid_pf;
        __syncthreads();                 // stage visible; the other stage's readers finished a tile ago
        const int next = tile + 1 < tend ? tile + 1 : -1;
        if (next >= 0) {
            const u32x4* g = reinterpret_cast<const u32x4*>(Bc + static_cast<size_t>(next) * 32 * kpad);
#pragma unroll
            for (int u = 0; u < PF; ++u) {
                const int ch = threadIdx.x + u * 64 * WV;
                if (ch < CHUNKS) pf[u] = g[ch];
            }
            if constexpr (LEARNED) cid_pf = ba.cid[static_cast<size_t>(next) * 32 + (lane & 31)];
        }
        // all fragment reads are issued before the products (up to 16 at a
        // time), and even / odd K-steps go to two accumulators, so the chain of
        // dependent MFMAs is half as long and does not wait on each LDS read
        f32x16 acc;
        {
            constexpr int BATCH = KS <= 16 ? KS : 4;
            const f32x16 zero = {};
            f32x16 acc0 = zero, acc1 = zero;
#pragma unroll
            for (int s0 = 0; s0 < KS; s0 += BATCH) {
                frag bfr[BATCH];
#pragma unroll
                for (int u = 0; u < BATCH; ++u)
                    if (s0 + u < KS) bfr[u] = s_tile[stage][s0 + u][half][lane & 31];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < BATCH; ++u) {
                    const int s = s0 + u;
                    if (s < KS) {
                        if (s % 2 == 0)
                            acc0 = Tr::mma(qa[s], bfr[u], acc0);
                        else
                            acc1 = Tr::mma(qa[s], bfr[u], acc1);
                    }
                }
            }
            acc = KS > 1 ? acc0 + acc1 : acc0;
        }

        const int cand = LEARNED ? cid_cur : tile * 32 + (lane & 31);
        const bool valid = LEARNED ? cand >= 0 : cand < n;
        pairs += static_cast<unsigned long long>(nq_valid) *
                 static_cast<unsigned long long>(__popcll(__ballot(valid) & 0xFFFFFFFFull));
        if (filling) {
            // the first CAP / 32 tiles go straight into the (empty) lists
            const int slot = it * 32 + (lane & 31);
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (qrow[r] >= 0)
                    lists[static_cast<size_t>(qrow[r]) * CAP + slot] =
                        valid ? make_key(acc[r], static_cast<uint32_t>(cand)) : KEY_INF;
            if (it + 1 == fill_tiles || next < 0) {
                filling = false;
                // the lists' stores complete before other lanes read them
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                for (int q = 0; q < NQ; ++q) {
                    const int qg = s_qid[wave][q];
                    if (qg < 0) continue;
                    const float nt = sort_query_list<E>(lists + static_cast<size_t>(qg) * CAP, kp);
                    const int rr = 4 * (q / 8) + (q % 4), hh = (q / 4) & 1;
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (r == rr && half == hh) tauv[r] = nt;
                }
            }
            tile = next;
            continue;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float sc = acc[r];
            uint64_t mask = __ballot(valid && sc <= tauv[r]);
            if (mask) {
                const int qa_ = acc_row(r, 0), qb_ = acc_row(r, 1);
                uint32_t ma = static_cast<uint32_t>(mask), mb = static_cast<uint32_t>(mask >> 32);
                int ca = cnt_of(qa_), cb = cnt_of(qb_);
                const bool fa = ca + __popc(ma) > BUF, fb = cb + __popc(mb) > BUF;
                if (fa || fb) {
                    // a full buffer is merged before this tile's keys are added,
                    // so every merge takes nearly BUF keys
                    wave_lds_sync();
                    if (fa) {
                        const int qg = s_qid[wave][qa_];
                        float nt = -__uint_as_float(0x7F800000u);
                        if (qg >= 0)
                            nt = merge_query_list<E>(lists + static_cast<size_t>(qg) * CAP, &s_buf[wave][qa_][0], ca,
                                                     kp);
                        if (half == 0) tauv[r] = MODE == 2 ? fminf(tauv[r], nt) : nt;
                        ca = 0;
                        cntw[qa_ >> 2] &= ~(0xFFu << (8 * (qa_ & 3)));
                    }
                    if (fb) {
                        const int qg = s_qid[wave][qb_];
                        float nt = -__uint_as_float(0x7F800000u);
                        if (qg >= 0)
                            nt = merge_query_list<E>(lists + static_cast<size_t>(qg) * CAP, &s_buf[wave][qb_][0], cb,
                                                     kp);
                        if (half == 1) tauv[r] = MODE == 2 ? fminf(tauv[r], nt) : nt;
                        cb = 0;
                        cntw[qb_ >> 2] &= ~(0xFFu << (8 * (qb_ & 3)));
                    }
                    wave_lds_sync();
                    mask = __ballot(valid && sc <= tauv[r]);
                    ma = static_cast<uint32_t>(mask);
                    mb = static_cast<uint32_t>(mask >> 32);
                }
                // slot: the half's count plus the rank among the half's
                // passing lanes (mbcnt64 counts the lower half's lanes too in
                // the upper half)
                const int pa = __popc(ma), pb = __popc(mb);
                const int slot0 = half ? qb_ * BUF + cb - pa : qa_ * BUF + ca;
                if (valid && sc <= tauv[r])
                    (&s_buf[wave][0][0])[slot0 + mbcnt64(mask)] = make_key(sc, static_cast<uint32_t>(cand));
                cntw[qa_ >> 2] += static_cast<uint32_t>(pa) << (8 * (qa_ & 3));
                cntw[qb_ >> 2] += static_cast<uint32_t>(pb) << (8 * (qb_ & 3));
            }
        }
        tile = next;
    }
    wave_lds_sync();
    {
        // the last merges in a loop that is not unrolled: query q's count
        // moved to lane q
        int cnt_lane = 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            if (lane == q) cnt_lane = cnt_of(q);
        uint64_t nonempty = __ballot(cnt_lane > 0);
        while (nonempty) {
            const int q = __builtin_ctzll(nonempty);
            nonempty &= nonempty - 1;
            const int qg = s_qid[wave][q];
            if (qg >= 0)
                merge_query_list<E>(lists + static_cast<size_t>(qg) * CAP, &s_buf[wave][q][0],
                                    __builtin_amdgcn_readlane(cnt_lane, q), kp);
            wave_lds_sync();
        }
    }
    count_pairs(pair_count, pairs);

    if constexpr (LEARNED) return;
    // certificate lower bound for the candidates left out of each list
    const double R = static_cast<double>(__uint_as_float(*rmax_bits));
    if (lane < NQ) {
        const int qg = s_qid[wave][lane];
        if (qg >= 0) {
            float sl = key_dist(lists[static_cast<size_t>(qg) * CAP + (kp - 1)]);
            if (MODE == 2) sl = fminf(sl, lb_out[qg]);   // as in k_select_tree
            const double yi2 = static_cast<double>(ynorm2[qg]);
            const double yi = sqrt(yi2);
            const double Ei =
                em.gamma * (R + 1.05 * yi) * (R + 1.05 * yi) + em.norm * R * R + em.cross * yi * R + 1e-30;
            const double t = static_cast<double>(sl) + yi2 - Ei;
            double D = t > 0.0 ? sqrt(t) : 0.0;
            D -= em.center * (yi + R);
            D = D > 0.0 ? D : 0.0;
            lb_out[qg] = static_cast<float>(D * D * (1.0 - 1.0 / 1048576.0));
        }
    }
}

// ------------------------------------------------------------------ launchers
// The block partials go to colpart while they fit its colblocks rows, else (n >
// 128) to `room`: the query operand's n rows of at least 2 m bytes, written
// later, hold the ceil(n / 128) rows of 8 m bytes.
hipError_t launch_colmean(const float* X, int n, int m, double* colpart, int colblocks, void* room, double* mu,
                          hipStream_t st)
{
    const int nb = std::max(1, std::min(1024, (n + 127) / 128));
    const int rpb = (n + nb - 1) / nb;
    double* part = nb > colblocks ? static_cast<double*>(room) : colpart;
    hipLaunchKernelGGL(k_colsum_partial, dim3(nb), dim3(256), 0, st, X, n, m, rpb, part);
    hipLaunchKernelGGL(k_colsum_finish, dim3(m), dim3(WAVE), 0, st, part, nb, m, n, mu);
    return hipGetLastError();
}

// sample-order operand rows (no row maps): one thread per row for short rows
static void launch_rows(const float* X, int n, int npad, int m, const double* mu, int split, int kpad, void* Aq,
                        void* Bc, float* ynorm2, unsigned* rmax_bits, const int* brow, const int* arow, hipStream_t st)
{
    if (m <= PREP_THREAD_M && split == 0 && !brow && !arow)
        hipLaunchKernelGGL(k_prep_rows_thread, dim3((npad + 255) / 256), dim3(256), 0, st, X, n, npad, m, mu, split,
                           kpad, Aq, Bc, ynorm2, rmax_bits);
    else
        hipLaunchKernelGGL(k_prep_rows, dim3(prep_blocks(npad)), dim3(256), 0, st, X, n, npad, m, mu, split, kpad, Aq,
                           Bc, ynorm2, rmax_bits, brow, arow);
}

hipError_t launch_prep_rows(const float* X, int n, int m, const double* mu, int split, int kpad, void* Aq, void* Bc,
                            float* ynorm2, unsigned* rmax_bits, const int* brow, const int* arow, hipStream_t st)
{
    const int npad = brow ? n : (n + 31) / 32 * 32;
    launch_rows(X, n, npad, m, mu, split, kpad, Aq, Bc, ynorm2, rmax_bits, brow, arow, st);
    return hipGetLastError();
}

// Xs holds the samples in curve order, so operand row p is input row p: the
// sample-order kernels without row maps, reading and writing rows in order
hipError_t launch_prep_rows_curve(const float* Xs, int n, int m, const double* mu, int split, int kpad, void* Aq,
                                  void* Bc, float* ynorm2, unsigned* rmax_bits, hipStream_t st)
{
    const int npad = (n + 31) / 32 * 32;
    launch_rows(Xs, n, npad, m, mu, split, kpad, Aq, Bc, ynorm2, rmax_bits, nullptr, nullptr, st);
    return hipGetLastError();
}

hipError_t launch_prep(const float* X, int n, int m, int split, int kpad, double* colpart, int colblocks,
                       double* mu, void* Aq, void* Bc, float* ynorm2, unsigned* rmax_bits, const int* brow,
                       const int* arow, hipStream_t st)
{
    // with a row map the padding rows of the last tile are filled separately
    const int npad = brow ? n : (n + 31) / 32 * 32;
    const hipError_t e = launch_colmean(X, n, m, colpart, colblocks, Aq, mu, st);
    if (e != hipSuccess) return e;
    launch_rows(X, n, npad, m, mu, split, kpad, Aq, Bc, ynorm2, rmax_bits, brow, arow, st);
    return hipGetLastError();
}

template <class Tr, int KS, int WV>
static hipError_t launch_sel(const void* Aq, const void* Bc, int n, int kp, const float* ynorm2, const unsigned* rmax,
                             ErrModel em, uint64_t* lists, int cap, float* lb, const BucketArgs* ba, int max_work,
                             const CurveArgs* crv, unsigned long long* pairs, hipStream_t st)
{
    using elem = typename Tr::elem;
    const int rows_per_block = WV * 32;
    const dim3 block(64 * WV);
    const elem* A = static_cast<const elem*>(Aq);
    const elem* B = static_cast<const elem*>(Bc);
    // the lists buffer holds n * cap keys; only capacities 128 and 256 exist
    if (kp > cap) return hipErrorInvalidValue;
    if (cap != 128 && cap != 256) return hipErrorInvalidValue;
    const BucketArgs nb = {};
    if (ba) {
        if (max_work <= 0) return hipSuccess;
        const dim3 grid(max_work);
        if (cap == 128)
            hipLaunchKernelGGL((k_select_mfma<Tr, KS, WV, 2, 1>), grid, block, 0, st, A, B, n, kp, ynorm2, rmax, em,
                               lists, lb, *ba, nullptr, nullptr, pairs);
        else
            hipLaunchKernelGGL((k_select_mfma<Tr, KS, WV, 4, 1>), grid, block, 0, st, A, B, n, kp, ynorm2, rmax, em,
                               lists, lb, *ba, nullptr, nullptr, pairs);
        return hipGetLastError();
    }
    const dim3 grid((n + rows_per_block - 1) / rows_per_block);
    if (crv) {
        if (cap == 128)
            hipLaunchKernelGGL((k_select_mfma<Tr, KS, WV, 2, 2>), grid, block, 0, st, A, B, n, kp, ynorm2, rmax, em,
                               lists, lb, nb, crv->wide_count, crv->wide, pairs);
        else
            hipLaunchKernelGGL((k_select_mfma<Tr, KS, WV, 4, 2>), grid, block, 0, st, A, B, n, kp, ynorm2, rmax, em,
                               lists, lb, nb, crv->wide_count, crv->wide, pairs);
        return hipGetLastError();
    }
    if (cap == 128)
        hipLaunchKernelGGL((k_select_mfma<Tr, KS, WV, 2, 0>), grid, block, 0, st, A, B, n, kp, ynorm2, rmax, em, lists,
                           lb, nb, nullptr, nullptr, pairs);
    else
        hipLaunchKernelGGL((k_select_mfma<Tr, KS, WV, 4, 0>), grid, block, 0, st, A, B, n, kp, ynorm2, rmax, em, lists,
                           lb, nb, nullptr, nullptr, pairs);
    return hipGetLastError();
}

// Instantiated contraction lengths (in MFMA K-steps); the operand K is padded
// with zeros up to the next one. WV (wavefronts per workgroup) is 8 where the
// two LDS stages and the query buffers fit in LDS, else 4.
static const int kBf16Steps[] = {2, 3, 4, 5, 6, 7, 8, 10, 13, 16, 20, 25, 32};
static const int kF32Steps[] = {2, 4, 6, 8, 10, 12, 16, 24, 32, 48, 64, 96, 128};

int mfma_kstep(int split) { return split == 0 ? TraitsF32::KSTEP : TraitsBF16::KSTEP; }

int mfma_pick_ksteps(int split, int needed)
{
    const int* lst = split == 0 ? kF32Steps : kBf16Steps;
    const int cnt = split == 0 ? static_cast<int>(sizeof(kF32Steps) / sizeof(int))
                               : static_cast<int>(sizeof(kBf16Steps) / sizeof(int));
    for (int t = 0; t < cnt; ++t)
        if (lst[t] >= needed) return lst[t];
    return -1;
}

#define KVB_SEL_CASE(TR, K, WV) \
    case K: return launch_sel<TR, K, WV>(Aq, Bc, n, kp, ynorm2, rmax, em, lists, cap, lb, ba, max_work, crv, pairs, st);

int select_mfma_queries_per_block(int split, int kpad)
{
    const int ks = kpad / mfma_kstep(split);
    const bool four = split == 0 ? ks >= 64 : ks >= 32;
    return (four ? 4 : 8) * 32;
}

hipError_t launch_select_mfma(int split, const void* Aq, const void* Bc, int n, int kpad, int kp, const float* ynorm2,
                              const unsigned* rmax, ErrModel em, uint64_t* lists, int cap, float* lb,
                              const BucketArgs* ba, int max_work, const CurveArgs* crv, unsigned long long* pairs,
                              hipStream_t st)
{
    const int ks = kpad / mfma_kstep(split);
    if (split == 0) {
        switch (ks) {
            KVB_SEL_CASE(TraitsF32, 2, 8)
            KVB_SEL_CASE(TraitsF32, 4, 8)
            KVB_SEL_CASE(TraitsF32, 6, 8)
            KVB_SEL_CASE(TraitsF32, 8, 8)
            KVB_SEL_CASE(TraitsF32, 10, 8)
            KVB_SEL_CASE(TraitsF32, 12, 8)
            KVB_SEL_CASE(TraitsF32, 16, 8)
            KVB_SEL_CASE(TraitsF32, 24, 8)
            KVB_SEL_CASE(TraitsF32, 32, 8)
            KVB_SEL_CASE(TraitsF32, 48, 8)
            KVB_SEL_CASE(TraitsF32, 64, 4)
            KVB_SEL_CASE(TraitsF32, 96, 4)
            KVB_SEL_CASE(TraitsF32, 128, 4)
        default: return hipErrorInvalidValue;
        }
    }
    switch (ks) {
        KVB_SEL_CASE(TraitsBF16, 2, 8)
        KVB_SEL_CASE(TraitsBF16, 3, 8)
        KVB_SEL_CASE(TraitsBF16, 4, 8)
        KVB_SEL_CASE(TraitsBF16, 5, 8)
        KVB_SEL_CASE(TraitsBF16, 6, 8)
        KVB_SEL_CASE(TraitsBF16, 7, 8)
        KVB_SEL_CASE(TraitsBF16, 8, 8)
        KVB_SEL_CASE(TraitsBF16, 10, 8)
        KVB_SEL_CASE(TraitsBF16, 13, 8)
        KVB_SEL_CASE(TraitsBF16, 16, 8)
        KVB_SEL_CASE(TraitsBF16, 20, 8)
        KVB_SEL_CASE(TraitsBF16, 25, 8)
        KVB_SEL_CASE(TraitsBF16, 32, 4)
    default: return hipErrorInvalidValue;
    }
}
#undef KVB_SEL_CASE

}  // namespace kvb
