// Kernels of the learned partitioner's MLP (gfx950): BF16 MFMA GEMMs with
// fused epilogues, layout helpers, soft-target softmax cross-entropy, Adam,
// top-P routing and a counter-based generator for seeded parameters.
//
// Every GEMM here is C[M, N] = A[M, K] . B[N, K]^T with A and B row-major BF16
// (K contiguous), FP32 accumulation on v_mfma_f32_32x32x16_bf16, 32 x 32
// output tiles. M, N are multiples of 32 and K a
// multiple of 16 (the caller pads).
#include <algorithm>

#include <type_traits>

#include "kvb_device.h"
#include "kvb_kernels.h"

namespace kvb {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint16_t f2bf(float f)
{
    const uint32_t u = __float_as_uint(f);
    const uint32_t r = ((u >> 16) & 1u) + 0x7FFFu;
    return static_cast<uint16_t>((u + r) >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float(static_cast<uint32_t>(h) << 16); }

// Epilogue: v = acc (+ bias[col]); relu: v = max(v, 0); mask: v = 0 where
// mask_ref[row, col] <= 0; then optional float32, BF16 and transposed BF16
// (Ct [N, M]) stores. The four accumulator registers of a group hold four
// consecutive rows of one column, so the transposed copy takes one 8-byte
// store per group and the backward products need no transpose pass.
__device__ __forceinline__ void gemm_store4(const GemmJob& g, int row0, int col, float bcol, float (&v)[4])
{
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        v[u] += bcol;
        if (g.relu) v[u] = fmaxf(v[u], 0.f);
        if (g.mask_ref && g.mask_ref[static_cast<size_t>(row0 + u) * g.ldm + col] <= 0.f) v[u] = 0.f;
        if (g.Cf) g.Cf[static_cast<size_t>(row0 + u) * g.ldcf + col] = v[u];
        if (g.Cb) g.Cb[static_cast<size_t>(row0 + u) * g.ldcb + col] = f2bf(v[u]);
    }
    if (g.Ct) {
        uint2 t;
        t.x = f2bf(v[0]) | (static_cast<uint32_t>(f2bf(v[1])) << 16);
        t.y = f2bf(v[2]) | (static_cast<uint32_t>(f2bf(v[3])) << 16);
        *reinterpret_cast<uint2*>(g.Ct + static_cast<size_t>(col) * g.M + row0) = t;
    }
}

// acc + A tile . B tile^T over the k-steps s0 .. s1 - 1 (16 each), in order;
// the operands of eight steps are loaded together, so a short batch waits for
// memory once per eight steps instead of once per step.
__device__ __forceinline__ f32x16 gemm_steps(const uint16_t* ap, const uint16_t* bp, int s0, int s1, f32x16 acc)
{
    constexpr int U = 8;
    int s = s0;
    for (; s + U <= s1; s += U) {
        bf16x8 a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            a[u] = *reinterpret_cast<const bf16x8*>(ap + (s + u) * 16);
            b[u] = *reinterpret_cast<const bf16x8*>(bp + (s + u) * 16);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[u], b[u], acc, 0, 0, 0);
    }
    for (; s < s1; ++s)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(ap + s * 16),
                                                      *reinterpret_cast<const bf16x8*>(bp + s * 16), acc, 0, 0, 0);
    return acc;
}

// One wavefront per output tile, the k-steps in order (the forward products:
// the order of a logit's sum is part of the routing).
__global__ __launch_bounds__(256) void k_gemm_nt(GemmJob g)
{
    const int lane = lane_id();
    const int wave = threadIdx.x >> 6;
    const int tiles_n = g.N / 32;
    const int tile = blockIdx.x * 4 + wave;
    if (tile >= (g.M / 32) * tiles_n) return;
    const int m0 = (tile / tiles_n) * 32, n0 = (tile % tiles_n) * 32;
    const int half = lane >> 5;
    const uint16_t* ap = g.A + static_cast<size_t>(m0 + (lane & 31)) * g.lda + half * 8;
    const uint16_t* bp = g.B + static_cast<size_t>(n0 + (lane & 31)) * g.ldb + half * 8;
    const f32x16 zero = {};
    const f32x16 acc = gemm_steps(ap, bp, 0, g.K / 16, zero);
    const int col = n0 + (lane & 31);
    const float bcol = g.bias ? g.bias[col] : 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float v[4] = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        gemm_store4(g, m0 + 8 * q + 4 * half, col, bcol, v);
    }
}

// Two by two output tiles per wavefront, each sum in the order of k_gemm_nt: half
// the operand loads per product (the large forward products are bound by them).
// 32768 rows of 128-256-256-1024: 180 to 115 us in three launches.
__global__ __launch_bounds__(256) void k_gemm_nt_wide(GemmJob g)
{
    constexpr int U = 4;   // k-steps loaded together
    const int lane = lane_id();
    const int wave = threadIdx.x >> 6;
    const int tiles_n = g.N / 64;
    const int tile = blockIdx.x * 4 + wave;
    if (tile >= (g.M / 64) * tiles_n) return;
    const int m0 = (tile / tiles_n) * 64, n0 = (tile % tiles_n) * 64;
    const int half = lane >> 5;
    const uint16_t* ap = g.A + static_cast<size_t>(m0 + (lane & 31)) * g.lda + half * 8;
    const uint16_t* bp = g.B + static_cast<size_t>(n0 + (lane & 31)) * g.ldb + half * 8;
    const size_t a32 = static_cast<size_t>(32) * g.lda, b32 = static_cast<size_t>(32) * g.ldb;
    f32x16 acc[2][2] = {};
    auto steps = [&](auto count, int s) {
        constexpr int N = decltype(count)::value;
        bf16x8 a[N][2], b[N][2];
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                a[u][h] = *reinterpret_cast<const bf16x8*>(ap + h * a32 + (s + u) * 16);
                b[u][h] = *reinterpret_cast<const bf16x8*>(bp + h * b32 + (s + u) * 16);
            }
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int w = 0; w < 2; ++w)
                    acc[h][w] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[u][h], b[u][w], acc[h][w], 0, 0, 0);
    };
    const int ks = g.K / 16;
    int s = 0;
    for (; s + U <= ks; s += U) steps(std::integral_constant<int, U>{}, s);
    for (; s < ks; ++s) steps(std::integral_constant<int, 1>{}, s);
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const int col = n0 + 32 * w + (lane & 31);
        const float bcol = g.bias ? g.bias[col] : 0.f;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4] = {acc[h][w][4 * q], acc[h][w][4 * q + 1], acc[h][w][4 * q + 2], acc[h][w][4 * q + 3]};
                gemm_store4(g, m0 + 32 * h + 8 * q + 4 * half, col, bcol, v);
            }
    }
}

// One workgroup per output tile, the k-steps in four consecutive quarters, one
// per wavefront: the backward products of a training batch have few tiles (32
// to 256) and a long contraction, so their time is the chain of loads. All
// four wavefronts load their quarter at once; the accumulator then passes
// from wavefront to wavefront through LDS, so every sum keeps the order of
// k_gemm_nt. Two independent products share one launch (job 0: workgroups
// below tiles0). The backward products of a 512-row batch (128-256-256-1024):
// 53 us in five launches with one tile per wavefront and one load per step,
// 25 us in three launches now.
__global__ __launch_bounds__(256) void k_gemm_nt_split(GemmJob j0, GemmJob j1, int tiles0)
{
    constexpr int PRE = 16;   // steps a wavefront loads ahead of its turn
    __shared__ float s_acc[16][WAVE];
    const bool second = static_cast<int>(blockIdx.x) >= tiles0;
    const GemmJob& g = second ? j1 : j0;
    const int tile = blockIdx.x - (second ? tiles0 : 0);
    const int lane = lane_id();
    const int wave = threadIdx.x >> 6;
    const int tiles_n = g.N / 32;
    const int m0 = (tile / tiles_n) * 32, n0 = (tile % tiles_n) * 32;
    const int half = lane >> 5;
    const uint16_t* ap = g.A + static_cast<size_t>(m0 + (lane & 31)) * g.lda + half * 8;
    const uint16_t* bp = g.B + static_cast<size_t>(n0 + (lane & 31)) * g.ldb + half * 8;
    const int steps = g.K / 16;
    const int s0 = steps * wave / 4, s1 = steps * (wave + 1) / 4;
    bf16x8 a[PRE], b[PRE];
#pragma unroll
    for (int u = 0; u < PRE; ++u)
        if (s0 + u < s1) {
            a[u] = *reinterpret_cast<const bf16x8*>(ap + (s0 + u) * 16);
            b[u] = *reinterpret_cast<const bf16x8*>(bp + (s0 + u) * 16);
        }
    for (int turn = 0; turn < 4; ++turn) {
        if (wave == turn) {
            f32x16 acc = {};
            if (turn > 0)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] = s_acc[r][lane];
#pragma unroll
            for (int u = 0; u < PRE; ++u)
                if (s0 + u < s1) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[u], b[u], acc, 0, 0, 0);
            if (s0 + PRE < s1) acc = gemm_steps(ap, bp, s0 + PRE, s1, acc);
#pragma unroll
            for (int r = 0; r < 16; ++r) s_acc[r][lane] = acc[r];
        }
        __syncthreads();
    }
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = s_acc[4 * wave + u][lane];
    const int col = n0 + (lane & 31);
    gemm_store4(g, m0 + 8 * wave + 4 * half, col, g.bias ? g.bias[col] : 0.f, v);
}

// dst[c, r] = src[r, c] for a rows x cols BF16 matrix (32 x 32 LDS tiles), for
// one or two matrices (blockIdx.z) in one launch.
__global__ __launch_bounds__(256) void k_transpose_bf16(TransposeJob j0, TransposeJob j1)
{
    __shared__ uint16_t t[32][33];
    const TransposeJob& j = blockIdx.z ? j1 : j0;
    const uint16_t* __restrict__ src = j.src;
    uint16_t* __restrict__ dst = j.dst;
    const int rows = j.rows, cols = j.cols;
    const int bx = blockIdx.x * 32, by = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
    for (int q = ty; q < 32; q += 8) {
        const int r = by + q, c = bx + tx;
        t[q][tx] = (r < rows && c < cols) ? src[static_cast<size_t>(r) * cols + c] : static_cast<uint16_t>(0);
    }
    __syncthreads();
    for (int q = ty; q < 32; q += 8) {
        const int c = bx + q, r = by + tx;
        if (c < cols && r < rows) dst[static_cast<size_t>(c) * rows + r] = t[tx][q];
    }
}

// Rows of a float32 matrix [valid, cols] (optionally gathered through idx) to
// BF16 [rows, ldd]; columns cols..ldd-1 and rows valid..rows-1 are zero.
__global__ __launch_bounds__(256) void k_cast_rows_bf16(const float* __restrict__ src, int cols,
                                                        const int32_t* __restrict__ idx, int valid, int rows,
                                                        int ldd, uint16_t* __restrict__ dst)
{
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= static_cast<int64_t>(rows) * ldd) return;
    const int r = static_cast<int>(t / ldd), c = static_cast<int>(t % ldd);
    if (c >= cols || r >= valid) {
        dst[t] = 0;
        return;
    }
    const int sr = idx ? idx[r] : r;
    dst[t] = f2bf(src[static_cast<size_t>(sr) * cols + c]);
}

__global__ __launch_bounds__(256) void k_cast_bf16(const float* __restrict__ src, int64_t cnt,
                                                   uint16_t* __restrict__ dst)
{
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t < cnt) dst[t] = f2bf(src[t]);
}

// Bias gradients out[c] = sum_r src[r, c] (float64 accumulation) of up to three
// matrices, and the batch's mean loss, in one launch: job blockIdx.y, 16
// columns per workgroup and 16 row lanes per column (lane l adds rows l, l + 16,
// ...), then the lanes in order. One thread per column, 512 dependent loads
// each, took 122 us per matrix of a 512-row batch; all three and the loss take 3.7 us.
__global__ __launch_bounds__(256) void k_colsums(ColSumJobs jobs, const double* __restrict__ row_loss, int rows,
                                                 double scale, double* __restrict__ loss, int add)
{
    __shared__ double s_part[16][17];
    if (blockIdx.y == 3) {
        if (blockIdx.x > 0) return;
        double s = 0.0;
        for (int r = threadIdx.x; r < rows; r += 256) s += row_loss[r];
        s = wave_sum_f64(s);
        if ((threadIdx.x & 63) == 0) s_part[0][threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            const double t = (s_part[0][0] + s_part[0][1]) + (s_part[0][2] + s_part[0][3]);
            loss[0] = (add ? loss[0] : 0.0) + t * scale;
        }
        return;
    }
    const ColSumJob j = jobs.job[blockIdx.y];
    const int c0 = blockIdx.x * 16;
    if (c0 >= j.cols) return;   // whole workgroup; cols is a multiple of 32
    const int c = threadIdx.x & 15, l = threadIdx.x >> 4;
    double s = 0.0;
#pragma unroll 8
    for (int r = l; r < rows; r += 16) s += static_cast<double>(j.src[static_cast<size_t>(r) * j.cols + c0 + c]);
    s_part[l][c] = s;
    __syncthreads();
    if (threadIdx.x < 16) {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < 16; ++q) t += s_part[q][threadIdx.x];
        j.out[c0 + threadIdx.x] = static_cast<float>(t);
    }
}

// Soft-target cross-entropy, one workgroup per row of logits Z [B, NB] (one
// wavefront per row left a 512-row batch on 128 of 256 CUs: 16.5 -> 8.6 us):
// target t_b = (1/ks) #{r : lab[i, r] == b} (a histogram built in LDS);
// loss_i = logsumexp(z) - sum_b t_b z_b; dZ = (softmax(z) - t) / B (float32 and
// BF16 copies); row losses to row_loss. Dynamic LDS: NB ints.
__global__ __launch_bounds__(256) void k_softmax_xent(const float* __restrict__ Z, int B, int NB,
                                                      const int32_t* __restrict__ lab, int ks,
                                                      float* __restrict__ dZ, uint16_t* __restrict__ dZb,
                                                      double* __restrict__ row_loss)
{
    extern __shared__ int hist[];
    __shared__ float s_mx[4];
    __shared__ double s_se[4], s_tz[4];
    const int wave = threadIdx.x >> 6;
    const bool lead = (threadIdx.x & 63) == 0;
    const int i = blockIdx.x;
    for (int b = threadIdx.x; b < NB; b += 256) hist[b] = 0;
    __syncthreads();
    const int32_t* li = lab + static_cast<size_t>(i) * ks;
    for (int r = threadIdx.x; r < ks; r += 256) {
        const int b = li[r];
        if (b >= 0 && b < NB) atomicAdd(&hist[b], 1);
    }
    const float* z = Z + static_cast<size_t>(i) * NB;
    float mx = -INFINITY;
    for (int b = threadIdx.x; b < NB; b += 256) mx = fmaxf(mx, z[b]);
    mx = wave_max_f32(mx);
    if (lead) s_mx[wave] = mx;
    __syncthreads();   // the histogram and the wavefronts' maxima
    mx = fmaxf(fmaxf(s_mx[0], s_mx[1]), fmaxf(s_mx[2], s_mx[3]));
    double se = 0.0, tz = 0.0;
    for (int b = threadIdx.x; b < NB; b += 256) {
        se += exp(static_cast<double>(z[b]) - static_cast<double>(mx));
        tz += static_cast<double>(hist[b]) * static_cast<double>(z[b]);
    }
    se = wave_sum_f64(se);
    tz = wave_sum_f64(tz);
    if (lead) {
        s_se[wave] = se;
        s_tz[wave] = tz;
    }
    __syncthreads();
    se = (s_se[0] + s_se[1]) + (s_se[2] + s_se[3]);
    tz = ((s_tz[0] + s_tz[1]) + (s_tz[2] + s_tz[3])) / ks;
    const double lse = static_cast<double>(mx) + log(se);
    const double invB = 1.0 / B;
    for (int b = threadIdx.x; b < NB; b += 256) {
        const double p = exp(static_cast<double>(z[b]) - lse);
        const float g = static_cast<float>((p - static_cast<double>(hist[b]) / ks) * invB);
        dZ[static_cast<size_t>(i) * NB + b] = g;
        dZb[static_cast<size_t>(i) * NB + b] = f2bf(g);
    }
    if (threadIdx.x == 0) row_loss[i] = lse - tz;
}

// Adam on float32 master parameters with a BF16 shadow (bias-corrected moments).
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ p, const float* __restrict__ g,
                                              float* __restrict__ m1, float* __restrict__ m2, int64_t cnt, float lr,
                                              float b1, float b2, float eps, float c1, float c2,
                                              uint16_t* __restrict__ pb)
{
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= cnt) return;
    const float gt = g[t];
    const float a = b1 * m1[t] + (1.f - b1) * gt;
    const float v = b2 * m2[t] + (1.f - b2) * gt * gt;
    m1[t] = a;
    m2[t] = v;
    const float w = p[t] - lr * (a / c1) / (sqrtf(v / c2) + eps);
    p[t] = w;
    if (pb) pb[t] = f2bf(w);
}

// Top-P buckets of each logits row (descending value, ties to the smaller
// bucket id); home = the first. One wavefront per row, P rounds of a
// wavefront arg-max over the row with earlier winners excluded.
template <int PMAX>
__global__ __launch_bounds__(256) void k_route_topp(const float* __restrict__ Z, int rows, int NB, int P,
                                                    int32_t* __restrict__ home, int32_t* __restrict__ probe)
{
    const int lane = lane_id();
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= rows) return;
    const float* z = Z + static_cast<size_t>(i) * NB;
    int chosen[PMAX];
#pragma unroll
    for (int u = 0; u < PMAX; ++u) chosen[u] = -1;
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
        if (p < P) {
            float bv = -INFINITY;
            int bi = 0x7fffffff;
            for (int b = lane; b < NB; b += WAVE) {
                bool taken = false;
#pragma unroll
                for (int u = 0; u < PMAX; ++u) taken |= (chosen[u] == b);
                float v = z[b];
                if (v != v) v = -INFINITY;   // a NaN logit ranks last
                if (!taken && (v > bv || (v == bv && b < bi))) {
                    bv = v;
                    bi = b;
                }
            }
            for (int o = 32; o > 0; o >>= 1) {
                const float ov = __shfl_xor(bv, o, WAVE);
                const int oi = __shfl_xor(bi, o, WAVE);
                if (ov > bv || (ov == bv && oi < bi)) {
                    bv = ov;
                    bi = oi;
                }
            }
            chosen[p] = bi;
            if (lane == 0) probe[static_cast<size_t>(i) * P + p] = bi;
        }
    }
    if (lane == 0 && home) home[i] = chosen[0];
}

// The same for NB <= 64 NV: the row is read once, NV logits per lane in order
// bits (a taken one is 0, below every logit's), and a round takes the wavefront's
// maximum and, of the lanes that hold it, the smallest bucket. Bound by reading
// the logits; re-reading the row from the caches in every round took 130 us for
// 32768 rows of 1024 and four rounds, this 35 (3.8 TB/s).
template <int NV>
__global__ __launch_bounds__(256) void k_route_topp_row(const float* __restrict__ Z, int rows, int NB, int P,
                                                        int32_t* __restrict__ home, int32_t* __restrict__ probe)
{
    const int lane = lane_id();
    const int i = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (i >= rows) return;
    const float* z = Z + static_cast<size_t>(i) * NB;
    float raw[NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) raw[u] = z[min(u * WAVE + lane, NB - 1)];
    uint32_t v[NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) {
        float x = raw[u];
        if (x != x) x = -INFINITY;   // a NaN logit ranks last
        if (x == 0.f) x = 0.f;       // zeros of either sign tie
        v[u] = u * WAVE + lane < NB ? float_order_bits(x) : 0u;
    }
    for (int p = 0; p < P; ++p) {
        uint32_t bv = 0;
        int bu = 0;
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            bu = v[u] > bv ? u : bu;
            bv = max(bv, v[u]);
        }
        uint32_t top = bv;
#pragma unroll
        for (int o = 1; o < WAVE; o <<= 1) top = max(top, static_cast<uint32_t>(xor_lane(top, o)));
        const bool have = bv == top;
        uint64_t m = __ballot(have);
        int best = __builtin_amdgcn_readlane(bu * WAVE + lane, __builtin_ctzll(m));
        for (m &= m - 1; m; m &= m - 1)
            best = min(best, __builtin_amdgcn_readlane(bu * WAVE + lane, __builtin_ctzll(m)));
#pragma unroll
        for (int u = 0; u < NV; ++u)
            if (u * WAVE + lane == best) v[u] = 0u;
        if (lane == 0) {
            probe[static_cast<size_t>(i) * P + p] = best;
            if (p == 0 && home) home[i] = best;
        }
    }
}

// SplitMix64 (Steele, Lea and Flood; Vigna's constants) at counter c from seed,
// and a standard normal from two of its uniforms (Box-Muller).
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t c)
{
    uint64_t z = seed + (c + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
__device__ __forceinline__ double sm_normal(uint64_t seed, uint64_t c)
{
    const double u1 = (static_cast<double>(splitmix64(seed, 2 * c) >> 11) + 0.5) * (1.0 / 9007199254740992.0);
    const double u2 = static_cast<double>(splitmix64(seed, 2 * c + 1) >> 11) * (1.0 / 9007199254740992.0);
    return sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2);
}

// p[t] = scale * N(0, 1) draw number (offset + t) of the seeded stream.
__global__ __launch_bounds__(256) void k_fill_normal(float* __restrict__ p, int64_t cnt, uint64_t seed,
                                                     uint64_t offset, float scale)
{
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t < cnt) p[t] = scale * static_cast<float>(sm_normal(seed, offset + static_cast<uint64_t>(t)));
}

// ------------------------------------------------------------------ launchers
static bool gemm_ok(const GemmJob& g) { return g.M % 32 == 0 && g.N % 32 == 0 && g.K % 16 == 0; }
static int gemm_tiles(const GemmJob& g) { return (g.M / 32) * (g.N / 32); }

constexpr int GEMM_WIDE_MIN = 2048;
hipError_t launch_gemm_nt(const GemmJob& g, hipStream_t st)
{
    if (!gemm_ok(g)) return hipErrorInvalidValue;
    // two by two tiles each where that still leaves two wavefronts per SIMD (as
    // the products of 32768 routed rows do, 38 against 60 us; a training batch's
    // 32 to 256 tiles are one wavefront each, or k_gemm_nt_split)
    const int wide = g.M % 64 == 0 && g.N % 64 == 0 ? gemm_tiles(g) / 4 : 0;
    if (wide >= GEMM_WIDE_MIN)
        hipLaunchKernelGGL(k_gemm_nt_wide, dim3((wide + 3) / 4), dim3(256), 0, st, g);
    else
        hipLaunchKernelGGL(k_gemm_nt, dim3((gemm_tiles(g) + 3) / 4), dim3(256), 0, st, g);
    return hipGetLastError();
}

hipError_t launch_gemm_nt_split(const GemmJob& j0, const GemmJob* j1, hipStream_t st)
{
    if (!gemm_ok(j0) || (j1 && !gemm_ok(*j1))) return hipErrorInvalidValue;
    const int t0 = gemm_tiles(j0), t1 = j1 ? gemm_tiles(*j1) : 0;
    hipLaunchKernelGGL(k_gemm_nt_split, dim3(t0 + t1), dim3(256), 0, st, j0, j1 ? *j1 : j0, t0);
    return hipGetLastError();
}

hipError_t launch_transpose_bf16(const TransposeJob& j0, const TransposeJob* j1, hipStream_t st)
{
    const int rows = std::max(j0.rows, j1 ? j1->rows : 0), cols = std::max(j0.cols, j1 ? j1->cols : 0);
    hipLaunchKernelGGL(k_transpose_bf16, dim3((cols + 31) / 32, (rows + 31) / 32, j1 ? 2 : 1), dim3(256), 0, st, j0,
                       j1 ? *j1 : j0);
    return hipGetLastError();
}

hipError_t launch_cast_rows_bf16(const float* src, int cols, const int32_t* idx, int valid, int rows, int ldd,
                                 uint16_t* dst, hipStream_t st)
{
    const int64_t tot = static_cast<int64_t>(rows) * ldd;
    hipLaunchKernelGGL(k_cast_rows_bf16, dim3(static_cast<unsigned>((tot + 255) / 256)), dim3(256), 0, st, src, cols,
                       idx, valid, rows, ldd, dst);
    return hipGetLastError();
}

hipError_t launch_cast_bf16(const float* src, int64_t cnt, uint16_t* dst, hipStream_t st)
{
    hipLaunchKernelGGL(k_cast_bf16, dim3(static_cast<unsigned>((cnt + 255) / 256)), dim3(256), 0, st, src, cnt, dst);
    return hipGetLastError();
}

hipError_t launch_colsums(const ColSumJobs& jobs, const double* row_loss, int rows, double* loss, int add,
                          hipStream_t st)
{
    int cols = 0;
    for (const ColSumJob& j : jobs.job) {
        if (j.cols % 32) return hipErrorInvalidValue;
        cols = std::max(cols, j.cols);
    }
    hipLaunchKernelGGL(k_colsums, dim3(cols / 16, 4), dim3(256), 0, st, jobs, row_loss, rows, 1.0 / rows, loss, add);
    return hipGetLastError();
}

hipError_t launch_softmax_xent(const float* Z, int B, int NB, const int32_t* lab, int ks, float* dZ, uint16_t* dZb,
                               double* row_loss, hipStream_t st)
{
    hipLaunchKernelGGL(k_softmax_xent, dim3(B), dim3(256), NB * sizeof(int), st, Z, B, NB, lab, ks, dZ, dZb, row_loss);
    return hipGetLastError();
}

hipError_t launch_adam(float* p, const float* g, float* m1, float* m2, int64_t cnt, float lr, float b1, float b2,
                       float eps, float c1, float c2, uint16_t* pb, hipStream_t st)
{
    hipLaunchKernelGGL(k_adam, dim3(static_cast<unsigned>((cnt + 255) / 256)), dim3(256), 0, st, p, g, m1, m2, cnt, lr,
                       b1, b2, eps, c1, c2, pb);
    return hipGetLastError();
}

hipError_t launch_route_topp(const float* Z, int rows, int NB, int P, int32_t* home, int32_t* probe, hipStream_t st)
{
    if (P < 1 || P > 32 || P > NB) return hipErrorInvalidValue;
    // up to 1024 buckets a row fits the registers of a wavefront, 1, 4 or 16 logits
    // per lane (65536 rows of 32 buckets with their forward pass: 47 us with 1, 94 with 16, 77
    // by the wider rows' kernel; of 256: 94 with 4, 133, 162); wider rows are read again
    // in every round
    auto row = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((rows + 3) / 4), dim3(256), 0, st, Z, rows, NB, P, home, probe);
    };
    if (NB <= WAVE)
        row(k_route_topp_row<1>);
    else if (NB <= 4 * WAVE)
        row(k_route_topp_row<4>);
    else if (NB <= 16 * WAVE)
        row(k_route_topp_row<16>);
    else if (P <= 8)
        hipLaunchKernelGGL(k_route_topp<8>, dim3((rows + 3) / 4), dim3(256), 0, st, Z, rows, NB, P, home, probe);
    else
        hipLaunchKernelGGL(k_route_topp<32>, dim3((rows + 3) / 4), dim3(256), 0, st, Z, rows, NB, P, home, probe);
    return hipGetLastError();
}

hipError_t launch_fill_normal(float* p, int64_t cnt, uint64_t seed, uint64_t offset, float scale, hipStream_t st)
{
    hipLaunchKernelGGL(k_fill_normal, dim3(static_cast<unsigned>((cnt + 255) / 256)), dim3(256), 0, st, p, cnt, seed,
                       offset, scale);
    return hipGetLastError();
}

}  // namespace kvb
