// Leading eigenpairs of a symmetric CSR matrix (gfx950): Lanczos with full
// reorthogonalisation.
//
// The paper's use of the kernel matrix is spectral: the eigenpairs of the
// symmetric conjugate Lhat = e^{-1}(S^{-1} Kt S^{-1} - P^{-2}) (Section 2.2)
// approximate those of the Kolmogorov operator (Sections 2.2 and 5), and a
// sparse eigensolver is the most expensive step after the matrix itself
// (Section 4). Lhat is negative semi-definite; the wanted eigenvalues are the
// ones nearest zero, the top of its spectrum.
//
// Lanczos (Lanczos 1950; Golub and Van Loan, Section 10.1) builds an
// orthonormal basis v_0..v_{m-1} of the Krylov space of a seeded start vector
// with A v_j = beta_{j-1} v_{j-1} + alpha_j v_j + beta_j v_{j+1}. Rounding
// destroys the orthogonality as Ritz values converge, so every new vector is
// orthogonalised against all previous ones, twice (classical Gram-Schmidt
// repeated). The eigenpairs of the m x m tridiagonal T = tridiag(beta, alpha,
// beta) are the Ritz pairs; a Ritz vector is V s, its residual norm
// |beta_{m-1} s_{m-1}|. The small eigenproblem is solved on the host for the
// wanted pairs only: eigenvalues by bisection on the Sturm count, eigenvectors
// by inverse iteration (Golub and Van Loan, Sections 8.4 and 8.2).
//
// On the device: the matrix-vector product (16 lanes per row, FP64
// accumulation of float32 entries), the projections V^T w (one workgroup per
// four basis vectors and row chunk, then a fixed-order sum over the chunks),
// w -= V h (one thread per row), norms and Ritz vectors. Every reduction has a
// fixed order, so results are reproducible.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "kvb_ctx.h"
#include "kvb_device.h"

namespace kvb {

// y = A x, 16 lanes per row (four rows per wavefront): lane l takes entries l,
// l + 16, l + 32 and l + 48 of every 64, each in a sum of its own, and the sums
// are added in the order of a butterfly over 64 lanes. Bound by the gathers of
// x from L2; a wavefront per row of some 70 entries left most of its second
// pass idle (43 us at n = 100k and 6.9M entries, 39 us now).
__global__ __launch_bounds__(256) void k_spmv(const int64_t* __restrict__ rowptr, const int32_t* __restrict__ col,
                                              const float* __restrict__ val, const double* __restrict__ x, int n,
                                              double* __restrict__ y)
{
    constexpr int LPR = 16, Q = WAVE / LPR;
    const int sub = threadIdx.x % LPR;
    const int i = blockIdx.x * (256 / LPR) + threadIdx.x / LPR;
    double s[Q] = {};
    if (i < n) {
        const int64_t p1 = rowptr[i + 1];
        for (int64_t p = rowptr[i] + sub; p < p1; p += WAVE) {
            int c[Q];
            float v[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (p + q * LPR < p1) {
                    c[q] = col[p + q * LPR];
                    v[q] = val[p + q * LPR];
                }
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (p + q * LPR < p1) s[q] += static_cast<double>(v[q]) * x[c[q]];
        }
    }
    double t = (s[0] + s[2]) + (s[1] + s[3]);
#pragma unroll
    for (int o = LPR / 2; o > 0; o >>= 1) t += shfl_xor_f64(t, o);
    if (i < n && sub == 0) y[i] = t;
}

// part[s * ldp + c] = V[c][rows of chunk s] . w[same rows], PP_VECS columns per
// workgroup: they share the reads of w, and their loads overlap. Bound by
// reading V from the Infinity Cache (mean over the sweeps and norms of 400
// steps at n = 100k: 23.0 us with one column, 19.7 now). A few columns still
// spread over the whole chip; fixed-order reduction within each workgroup
// (wavefront butterflies, then the four wavefronts in order)
constexpr int PP_VECS = 4;
__global__ __launch_bounds__(256) void k_project_part(const double* __restrict__ V, int64_t ldv, int ncol,
                                                      const double* __restrict__ w, int n, int chunk, int ldp,
                                                      double* __restrict__ part)
{
    __shared__ double red[4][PP_VECS];
    const int c0 = blockIdx.x * PP_VECS;
    const double* v[PP_VECS];
#pragma unroll
    for (int u = 0; u < PP_VECS; ++u) v[u] = V + static_cast<size_t>(min(c0 + u, ncol - 1)) * ldv;
    const int64_t r0 = static_cast<int64_t>(blockIdx.y) * chunk;
    const int64_t r1 = r0 + chunk < n ? r0 + chunk : n;
    double s[PP_VECS] = {};
#pragma unroll 4
    for (int64_t r = r0 + threadIdx.x; r < r1; r += 256) {
        const double wr = w[r];
#pragma unroll
        for (int u = 0; u < PP_VECS; ++u) s[u] += v[u][r] * wr;
    }
#pragma unroll
    for (int u = 0; u < PP_VECS; ++u) {
        s[u] = wave_sum_f64(s[u]);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][u] = s[u];
    }
    __syncthreads();
    const int u = threadIdx.x;
    if (u < PP_VECS && c0 + u < ncol)
        part[static_cast<size_t>(blockIdx.y) * ldp + c0 + u] = (red[0][u] + red[1][u]) + (red[2][u] + red[3][u]);
}

// h[c] = sum over chunks s, in order, of part[s * ldp + c]; the last column's
// is alpha_j on the first Gram-Schmidt pass and is added to it on the second
__global__ __launch_bounds__(64) void k_project_sum(const double* __restrict__ part, int ncol, int nchunk, int ldp,
                                                    double* __restrict__ h, int first, double* __restrict__ alpha)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncol) return;
    double s = 0.0;
#pragma unroll 8
    for (int q = 0; q < nchunk; ++q) s += part[static_cast<size_t>(q) * ldp + c];
    h[c] = s;
    if (c == ncol - 1) *alpha = first ? s : *alpha + s;
}

// w[r] -= sum_c V[c][r] h[c]; one wavefront per workgroup, so that the last
// round of workgroups does not leave compute units idle
__global__ __launch_bounds__(64) void k_subtract_span(const double* __restrict__ V, int64_t ldv, int ncol,
                                                      const double* __restrict__ h, int n, double* __restrict__ w)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    double s = 0.0;
#pragma unroll 16
    for (int c = 0; c < ncol; ++c) s += V[static_cast<size_t>(c) * ldv + r] * h[c];
    w[r] -= s;
}

// out[r] = x[r] * scale
__global__ __launch_bounds__(256) void k_scale(const double* __restrict__ x, double scale, int n,
                                               double* __restrict__ out)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r < n) out[r] = x[r] * scale;
}

// b = sqrt(the sum over chunks, in order, of part[s * ldp]); out[r] = x[r] * (1 / b);
// the first thread stores b
__global__ __launch_bounds__(256) void k_scale_by_norm(const double* __restrict__ x, const double* __restrict__ part,
                                                       int nchunk, int ldp, int n, double* __restrict__ out,
                                                       double* __restrict__ b)
{
    double nrm2 = 0.0;
#pragma unroll 8
    for (int q = 0; q < nchunk; ++q) nrm2 += part[static_cast<size_t>(q) * ldp];
    const double bj = sqrt(nrm2);
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r == 0) b[0] = bj;
    if (r < n) out[r] = x[r] * (1.0 / bj);
}

// the seeded start vector: SplitMix64 (Steele, Lea and Flood 2014) of
// seed + r mapped to [-1, 1)
__global__ __launch_bounds__(256) void k_start_vector(uint64_t seed, int n, double* __restrict__ v)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    uint64_t z = seed + 0x9E3779B97F4A7C15ull * (static_cast<uint64_t>(r) + 1);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    v[r] = static_cast<double>(z >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

// Y[i][r] = sum_c V[c][r] S[c][i] (Ritz vectors), S as S[c * nev + i]. A
// workgroup forms RITZ_VECS vectors of its rows from one sweep of V (one vector
// at a time read V nev times: 5.8 ms for 36 vectors at n = 100k and 400
// columns, 0.31 ms now). Sums past the last vector are formed for nothing, and many
// sums leave few wavefronts: at 4, 8, 12, 16 and 24 vectors 424, 358, 304, 365 and 495 us
// there; 10 vectors of 128 columns 51, 50, 65, 79, 104, 25 113, 102, 86, 102, 146; n = 1M, 100
// columns, 8 vectors 305, 162, 224, 252, 321 and 64 2417, 1327, 1269, 971, 973. Eight
// and twelve are within 1.4 times the best of them everywhere, the others are not.
constexpr int RITZ_VECS = 12;
__global__ __launch_bounds__(256) void k_ritz(const double* __restrict__ V, int64_t ldv, int m,
                                              const double* __restrict__ S, int nev, int n, double* __restrict__ Y)
{
    const int r = min(static_cast<int>(blockIdx.x * blockDim.x + threadIdx.x), n - 1);
    const int i0 = blockIdx.y * RITZ_VECS;
    double s[RITZ_VECS] = {};
#pragma unroll 4
    for (int c = 0; c < m; ++c) {
        const double v = V[static_cast<size_t>(c) * ldv + r];
#pragma unroll
        for (int u = 0; u < RITZ_VECS; ++u)
            s[u] += v * S[static_cast<size_t>(c) * nev + min(i0 + u, nev - 1)];
    }
    if (static_cast<int>(blockIdx.x * blockDim.x + threadIdx.x) < n)
#pragma unroll
        for (int u = 0; u < RITZ_VECS; ++u)
            if (i0 + u < nev) Y[static_cast<size_t>(i0 + u) * n + r] = s[u];
}

// Spectral solution of the Kolmogorov problem (Section 3.1): with unit
// eigenvectors y_j of Lhat and S = P D^{1/2},
//   t = S g;  c_j = y_j . t;  f = S^{-1} sum_j y_j c_j / lambda_j;  g_l = S^{-1} sum_j y_j c_j.

// part[(q nvec + j) nchunk + s] = y_j . (S x_q) over the rows of chunk s (without
// WEIGHT: y_j . x_q), for RHS vectors x_0, x_1. Bound by reading Y once. A
// workgroup takes SP_VECS basis vectors and one row chunk, so the weights and
// the right sides are formed once per SP_VECS vectors, both right sides share
// one read of Y, and nvec / SP_VECS x nchunk workgroups (nchunk up to 64)
// cover the chip; one workgroup per vector over all rows left 36 of 256 CUs
// busy at 36 vectors (106 us per projection at n = 100k,
// 10 now for one right side and 12 for two).
// Fixed order: the threads' strided sums, wavefront butterflies, the four
// wavefronts, then the chunks (project_total).
constexpr int SP_VECS = 4;
template <int RHS, bool WEIGHT>
__global__ __launch_bounds__(256) void k_project_chunk(const double* __restrict__ Y, int nvec,
                                                       const double* __restrict__ x0, const double* __restrict__ x1,
                                                       const double* __restrict__ P, const double* __restrict__ D,
                                                       int n, int chunk, double* __restrict__ part)
{
    __shared__ double red[4][RHS * SP_VECS];
    const int j0 = blockIdx.x * SP_VECS;
    // 64 bits: the last chunk's end, and a thread's row past it, may lie beyond 2^31
    const int64_t r0 = static_cast<int64_t>(blockIdx.y) * chunk;
    const int64_t r1 = r0 + chunk < n ? r0 + chunk : n;
    const double* y[SP_VECS];
#pragma unroll
    for (int v = 0; v < SP_VECS; ++v) y[v] = Y + static_cast<size_t>(min(j0 + v, nvec - 1)) * n;
    double acc[RHS][SP_VECS] = {};
#pragma unroll 2
    for (int64_t r = r0 + threadIdx.x; r < r1; r += 256) {
        const double s = WEIGHT ? P[r] * sqrt(D[r]) : 1.0;
        const double w0 = WEIGHT ? s * x0[r] : x0[r];
        const double w1 = RHS > 1 ? (WEIGHT ? s * x1[r] : x1[r]) : 0.0;
#pragma unroll
        for (int v = 0; v < SP_VECS; ++v) {
            const double t = y[v][r];
            acc[0][v] += t * w0;
            if (RHS > 1) acc[RHS - 1][v] += t * w1;
        }
    }
#pragma unroll
    for (int q = 0; q < RHS; ++q)
#pragma unroll
        for (int v = 0; v < SP_VECS; ++v) {
            const double t = wave_sum_f64(acc[q][v]);
            if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][q * SP_VECS + v] = t;
        }
    __syncthreads();
    if (threadIdx.x < RHS * SP_VECS) {
        const int q = threadIdx.x / SP_VECS, j = j0 + threadIdx.x % SP_VECS, e = threadIdx.x;
        if (j < nvec)
            part[(static_cast<size_t>(q) * nvec + j) * gridDim.y + blockIdx.y] =
                (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]);
    }
}

// y_j . (S x_q) from its chunks (at most 64), one wavefront per (q, j).
__device__ __forceinline__ double project_total(const double* __restrict__ part, int nchunk, int qj)
{
    const int lane = lane_id();
    return wave_sum_f64(lane < nchunk ? part[static_cast<size_t>(qj) * nchunk + lane] : 0.0);
}

// cg_j = c_j, cf_j = c_j / lambda_j, and c_j to the host (lam, c_host: pinned)
__global__ __launch_bounds__(256) void k_solve_coef(const double* __restrict__ part, int nchunk, int nvec,
                                                    const double* __restrict__ lam, double* __restrict__ cf,
                                                    double* __restrict__ cg, double* __restrict__ c_host)
{
    const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (j >= nvec) return;
    const double c = project_total(part, nchunk, j);
    if (lane_id() == 0) {
        cg[j] = c;
        cf[j] = c / lam[j];
        c_host[j] = c;
    }
}

// coef = p, lambda p, q, lambda q (nvec each) from the projections p, q of two right sides
__global__ __launch_bounds__(256) void k_cdc_coef(const double* __restrict__ part, int nchunk, int nvec,
                                                  const double* __restrict__ lam, double* __restrict__ coef)
{
    const int qj = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (qj >= 2 * nvec) return;
    const double c = project_total(part, nchunk, qj);
    const int q = qj / nvec, j = qj % nvec;
    if (lane_id() == 0) {
        coef[(2 * q) * nvec + j] = c;
        coef[(2 * q + 1) * nvec + j] = lam[j] * c;
    }
}

// expansion coefficient of phi_l in grad u . grad v, in the y basis: (lambda_l a_l - b_l) / 2
__global__ __launch_bounds__(256) void k_cdc_grad_coef(const double* __restrict__ part, int nchunk, int nvec,
                                                       const double* __restrict__ lam, double* __restrict__ coef)
{
    const int l = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (l >= nvec) return;
    const double a = project_total(part, nchunk, l);
    const double b = project_total(part, nchunk, nvec + l);
    if (lane_id() == 0) coef[l] = 0.5 * (lam[l] * a - b);
}

__global__ __launch_bounds__(256) void k_expand(const double* __restrict__ Y, int nvec, const double* __restrict__ cf,
                                                const double* __restrict__ cg, const double* __restrict__ P,
                                                const double* __restrict__ D, int n, double* __restrict__ f,
                                                double* __restrict__ gl)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    double sf = 0.0, sg = 0.0;
#pragma unroll 8
    for (int j = 0; j < nvec; ++j) {
        const double y = Y[static_cast<size_t>(j) * n + r];
        sf += y * cf[j];
        sg += y * cg[j];
    }
    const double is = 1.0 / (P[r] * sqrt(D[r]));
    f[r] = sf * is;
    if (gl) gl[r] = sg * is;
}

// Carre du champ (Section 3.2): with p_j = y_j . S u and q_j = y_j . S v,
//   U = S^{-1} sum_j p_j y_j,  LU = S^{-1} sum_j lambda_j p_j y_j  (and V, LV from q),
//   t1 = S U V,  t2 = S (LU V + U LV).
__global__ __launch_bounds__(256) void k_cdc_products(const double* __restrict__ Y, int nvec,
                                                      const double* __restrict__ coef, const double* __restrict__ P,
                                                      const double* __restrict__ D, int n, double* __restrict__ t1,
                                                      double* __restrict__ t2)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    // coef: p, lambda p, q, lambda q (nvec each)
    double U = 0.0, LU = 0.0, V = 0.0, LV = 0.0;
#pragma unroll 8
    for (int j = 0; j < nvec; ++j) {
        const double y = Y[static_cast<size_t>(j) * n + r];
        U += coef[j] * y;
        LU += coef[nvec + j] * y;
        V += coef[2 * nvec + j] * y;
        LV += coef[3 * nvec + j] * y;
    }
    const double S = P[r] * sqrt(D[r]), is = 1.0 / S;
    U *= is;
    LU *= is;
    V *= is;
    LV *= is;
    t1[r] = S * U * V;
    t2[r] = S * (LU * V + U * LV);
}

// C[l][j][k] = <phi_l, phi_j phi_k>_S = sqrt(n) sum_r y_l y_j y_k / S_r for j <= k
// (one workgroup per pair (j, k), all l at once; the tensor is symmetric)
constexpr int CDC_MAX = 64;
__global__ __launch_bounds__(256) void k_cdc_tensor(const double* __restrict__ Y, int nvec,
                                                    const double* __restrict__ P, const double* __restrict__ D, int n,
                                                    const int* __restrict__ pair_j, const int* __restrict__ pair_k,
                                                    double* __restrict__ C)
{
    __shared__ double red[4][CDC_MAX];
    const int j = pair_j[blockIdx.x], k = pair_k[blockIdx.x];
    double acc[CDC_MAX];
#pragma unroll
    for (int l = 0; l < CDC_MAX; ++l) acc[l] = 0.0;
    for (int64_t r = threadIdx.x; r < n; r += 256) {
        const double w = Y[static_cast<size_t>(j) * n + r] * Y[static_cast<size_t>(k) * n + r] / (P[r] * sqrt(D[r]));
#pragma unroll
        for (int l = 0; l < CDC_MAX; ++l)
            if (l < nvec) acc[l] += Y[static_cast<size_t>(l) * n + r] * w;
    }
    const double rn = sqrt(static_cast<double>(n));
#pragma unroll
    for (int l = 0; l < CDC_MAX; ++l) {
        const double s = wave_sum_f64(acc[l]);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][l] = s;
    }
    __syncthreads();
    // each sorted triple l <= j <= k is written, with its permutations, by the
    // one workgroup of the pair (j, k), so every entry has a single writer
    for (int l = threadIdx.x; l <= j; l += 256) {
        const double v = ((red[0][l] + red[1][l]) + (red[2][l] + red[3][l])) * rn;
        const size_t nv = static_cast<size_t>(nvec);
        C[(l * nv + j) * nv + k] = v;
        C[(l * nv + k) * nv + j] = v;
        C[(j * nv + l) * nv + k] = v;
        C[(j * nv + k) * nv + l] = v;
        C[(k * nv + l) * nv + j] = v;
        C[(k * nv + j) * nv + l] = v;
    }
}

// Particle update of the density-evolution example (Section 5.3, explicit
// step of the sample SDE): x' = x + dt (u - grad f) + sqrt(dt) sigma w, with
// x, x' [n, m] float32 row-major, u and w [n, m] float64 row-major (or null:
// zero), grad [m, n] float64 (one gradient component per row).
__global__ __launch_bounds__(256) void k_advect(const float* __restrict__ X, int n, int m,
                                                const double* __restrict__ u, const double* __restrict__ grad,
                                                const double* __restrict__ w, double dt, double sdt,
                                                float* __restrict__ Xo)
{
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= static_cast<int64_t>(n) * m) return;
    const int r = static_cast<int>(t / m), s = static_cast<int>(t - static_cast<int64_t>(r) * m);
    double v = -grad[static_cast<size_t>(s) * n + r];
    if (u) v += u[t];
    double x = static_cast<double>(X[t]) + dt * v;
    if (w) x += sdt * w[t];
    Xo[t] = static_cast<float>(x);
}

}  // namespace kvb

namespace {

// Row chunks of the spectral projections: at least 512 rows each, at most 64
// (one wavefront adds them), and few enough that nvec sums per chunk fit in
// the n doubles a right side would take; one chunk writes its sums in place.
struct RowChunks {
    int rows, count;
};

RowChunks row_chunks(int n, int nvec)
{
    const int64_t want = std::max(1, std::min({64, n / 512, n / nvec}));
    const int64_t rows = (n + want - 1) / want;
    return {static_cast<int>(rows), static_cast<int>((n + rows - 1) / rows)};
}

// split of the Lanczos projections over rows: chunks of at least 8192 rows,
// at most 64 chunks
constexpr int PROJ_MIN_CHUNK = 8192;
constexpr int PROJ_MAX_CHUNKS = 64;

using namespace kvbh;

// Number of eigenvalues of the symmetric tridiagonal T = tridiag(b, a, b)
// below x: the negative pivots of the LDL^T factorisation of T - x I
// (Sylvester's law of inertia; the Sturm sequence count).
int count_below(const std::vector<double>& a, const std::vector<double>& b, int m, double x, double tiny)
{
    int c = 0;
    double q = a[0] - x;
    if (q == 0.0) q = -tiny;
    c += q < 0.0;
    for (int i = 1; i < m; ++i) {
        q = a[i] - x - b[i - 1] * b[i - 1] / q;
        if (q == 0.0) q = -tiny;
        c += q < 0.0;
    }
    return c;
}

// Solve (T - theta I) y = rhs in place: Gaussian elimination with partial
// pivoting on the tridiagonal band (row swaps fill one extra superdiagonal).
void shifted_solve(const std::vector<double>& a, const std::vector<double>& b, int m, double theta, double tiny,
                   std::vector<double>& y)
{
    std::vector<double> lo(m, 0.0), d(m), up(m, 0.0), up2(m, 0.0);
    std::vector<char> swapped(m, 0);
    for (int i = 0; i < m; ++i) d[i] = a[i] - theta;
    for (int i = 0; i + 1 < m; ++i) {
        lo[i] = b[i];
        up[i] = b[i];
    }
    for (int i = 0; i + 1 < m; ++i) {
        if (std::fabs(d[i]) >= std::fabs(lo[i])) {
            if (d[i] == 0.0) d[i] = tiny;
            const double f = lo[i] / d[i];
            lo[i] = f;
            d[i + 1] -= f * up[i];
        } else {
            // rows i and i + 1 trade places; row i + 1's entries move up
            const double f = d[i] / lo[i];
            d[i] = lo[i];
            lo[i] = f;
            const double u = up[i];
            up[i] = d[i + 1];
            d[i + 1] = u - f * d[i + 1];
            if (i + 2 < m) {
                up2[i] = up[i + 1];
                up[i + 1] = -f * up[i + 1];
            }
            swapped[i] = 1;
        }
    }
    if (d[m - 1] == 0.0) d[m - 1] = tiny;
    for (int i = 0; i + 1 < m; ++i) {
        if (swapped[i]) {
            const double t = y[i];
            y[i] = y[i + 1];
            y[i + 1] = t - lo[i] * y[i + 1];
        } else {
            y[i + 1] -= lo[i] * y[i];
        }
    }
    y[m - 1] /= d[m - 1];
    if (m > 1) y[m - 2] = (y[m - 2] - up[m - 2] * y[m - 1]) / d[m - 2];
    for (int i = m - 3; i >= 0; --i) y[i] = (y[i] - up[i] * y[i + 1] - up2[i] * y[i + 2]) / d[i];
}

// The nev largest eigenpairs of T (descending): each eigenvalue by bisection
// on the Sturm count to the resolution of double precision, its eigenvector
// by inverse iteration (three solves with T - theta I), orthogonalised against
// the vectors of nearby eigenvalues already found.
void top_eigenpairs(const std::vector<double>& a, const std::vector<double>& b, int m, int nev,
                    std::vector<double>& theta, std::vector<double>& Y)
{
    double lo = a[0], hi = a[0], norm = 0.0;
    for (int i = 0; i < m; ++i) {
        const double r = (i > 0 ? std::fabs(b[i - 1]) : 0.0) + (i + 1 < m ? std::fabs(b[i]) : 0.0);
        lo = std::min(lo, a[i] - r);
        hi = std::max(hi, a[i] + r);
        norm = std::max(norm, std::fabs(a[i]) + r);
    }
    const double tiny = 1e-300 + 2.2e-16 * norm;
    theta.assign(nev, 0.0);
    Y.assign(size_t(nev) * m, 0.0);
    for (int q = 0; q < nev; ++q) {
        const int idx = m - 1 - q;   // ascending rank of the wanted eigenvalue
        double l = lo, h = hi;
        for (int it = 0; it < 2000 && h - l > 4.4e-16 * std::max(std::fabs(l), std::fabs(h)) + 1e-300; ++it) {
            const double mid = 0.5 * (l + h);
            if (mid <= l || mid >= h) break;
            if (count_below(a, b, m, mid, tiny) > idx)
                h = mid;
            else
                l = mid;
        }
        theta[q] = 0.5 * (l + h);
        std::vector<double> y(m);
        double y0 = 0.0;
        for (int i = 0; i < m; ++i) {
            y[i] = 1.0 + 0.01 * std::sin(1.0 + 7.0 * i + 3.0 * q);
            y0 += y[i] * y[i];
        }
        y0 = std::sqrt(y0);
        for (int i = 0; i < m; ++i) y[i] /= y0;
        for (int it = 0; it < 3; ++it) {
            const std::vector<double> prev = y;
            shifted_solve(a, b, m, theta[q], tiny, y);
            for (int p = 0; p < q; ++p) {
                if (std::fabs(theta[p] - theta[q]) > 1e-3 * norm) continue;
                double dot = 0.0;
                for (int i = 0; i < m; ++i) dot += Y[size_t(p) * m + i] * y[i];
                for (int i = 0; i < m; ++i) y[i] -= dot * Y[size_t(p) * m + i];
            }
            // normalise after scaling by the largest entry: a pivot at the
            // floor (T - theta I exactly singular, as for T = 0) makes the
            // entries as large as 1/tiny, whose squares would overflow
            double amax = 0.0;
            for (int i = 0; i < m; ++i) amax = std::max(amax, std::fabs(y[i]));
            if (!(amax > 0.0) || !std::isfinite(amax)) {
                y = prev;   // keep the last unit iterate
                break;
            }
            double nrm = 0.0;
            for (int i = 0; i < m; ++i) {
                y[i] /= amax;
                nrm += y[i] * y[i];
            }
            nrm = std::sqrt(nrm);
            for (int i = 0; i < m; ++i) y[i] /= nrm;
        }
        for (int i = 0; i < m; ++i) Y[size_t(q) * m + i] = y[i];
    }
}

}  // namespace

extern "C" {

int kvb_lanczos_prefix(const double* alpha_host, const double* beta_host, int32_t ncv, int32_t* m_host)
{
    if (!alpha_host || !beta_host || !m_host || ncv < 1) return KVB_E_INVALID;
    // the steps up to the first breakdown (beta_j = 0 up to underflow: an
    // invariant subspace) or all ncv of them; every coefficient used must be
    // finite, and a NaN beta is not a breakdown
    int32_t m = 0;
    for (int32_t j = 0; j < ncv; ++j) {
        const double a = alpha_host[j], b = beta_host[j];
        *m_host = m;
        if (!std::isfinite(a) || !std::isfinite(b) || b < 0.0) return KVB_E_INVALID;
        m = j + 1;
        if (b <= 1e-300) break;
    }
    *m_host = m;
    return KVB_OK;
}

int kvb_eigsh(kvb_ctx ctx, const int64_t* rowptr, const int32_t* col, const float* val, int64_t n, int64_t nnz,
              int32_t nev, int32_t ncv, double tol, uint64_t seed, double* evals_host, double* resid_host,
              double* evecs)
{
    if (!ctx) return KVB_E_INVALID;
    KVB_REQUIRE(ctx, n >= 1 && n < (int64_t(1) << 31), "n must be in [1, 2^31)");
    KVB_REQUIRE(ctx, nev >= 1 && ncv >= nev && ncv <= 4096 && ncv <= n, "need 1 <= nev <= ncv <= min(4096, n)");
    KVB_REQUIRE(ctx, tol > 0 && std::isfinite(tol), "tol must be finite and > 0");
    KVB_REQUIRE(ctx, aligned(val), "val must be a non-null float32 device pointer");
    KVB_REQUIRE(ctx, evals_host != nullptr, "evals_host must be non-null");
    KVB_REQUIRE(ctx, evecs == nullptr || aligned(evecs), "evecs must be aligned");
    KVB_TRY(check_pattern(ctx, rowptr, col, n, nnz));
    const int nn = static_cast<int>(n);
    const int64_t ldv = (n + 63) / 64 * 64;
    const size_t need = round256(size_t(ncv + 1) * ldv * sizeof(double)) + round256(size_t(ldv) * sizeof(double)) +
                        round256(size_t(ncv + 1) * sizeof(double)) +
                        round256(size_t(ncv) * nev * sizeof(double)) +
                        round256(size_t(PROJ_MAX_CHUNKS) * (ncv + 1) * sizeof(double)) +
                        round256(2 * size_t(ncv) * sizeof(double)) + 2048;
    int rc = ensure_scratch(ctx, need);
    if (rc) return rc;
    Carve cv(ctx->scratch);
    double* V = cv.take<double>(size_t(ncv + 1) * ldv);
    double* w = cv.take<double>(ldv);
    double* h = cv.take<double>(ncv + 1);
    double* S = cv.take<double>(size_t(ncv) * nev);
    const int ldp = ncv + 1;
    double* part = cv.take<double>(size_t(PROJ_MAX_CHUNKS) * ldp);
    hipStream_t st = ctx->stream;
    const dim3 blk(256), rows_grid((nn + 255) / 256), spmv_grid((nn + 15) / 16);
    double* ab = cv.take<double>(2 * size_t(ncv));   // alpha_0..alpha_{ncv-1}, then beta_0..beta_{ncv-1}
    // row chunks of the projections: at least PROJ_MIN_CHUNK rows, a multiple
    // of 256, at most PROJ_MAX_CHUNKS of them
    int chunk = std::max(PROJ_MIN_CHUNK, (nn + PROJ_MAX_CHUNKS - 1) / PROJ_MAX_CHUNKS);
    chunk = (chunk + 255) / 256 * 256;
    const int nchunk = (nn + chunk - 1) / chunk;

    // part = the chunk sums of B[:, :ncol]^T x
    auto project = [&](const double* B, const double* x, int ncol) {
        hipLaunchKernelGGL(kvb::k_project_part, dim3((ncol + kvb::PP_VECS - 1) / kvb::PP_VECS, nchunk), blk, 0, st, B,
                           ldv, ncol, x, nn, chunk, ldp, part);
    };

    hipLaunchKernelGGL(kvb::k_start_vector, rows_grid, blk, 0, st, seed, nn, w);
    double b0 = 0.0;
    project(w, w, 1);
    hipLaunchKernelGGL(kvb::k_project_sum, dim3(1), dim3(64), 0, st, part, 1, nchunk, ldp, h, 1, ab);
    KVB_HIP(ctx, hipMemcpyAsync(&b0, h, sizeof(double), hipMemcpyDeviceToHost, st));
    KVB_HIP(ctx, hipStreamSynchronize(st));
    b0 = std::sqrt(b0);
    KVB_REQUIRE(ctx, b0 > 0, "start vector vanished");
    hipLaunchKernelGGL(kvb::k_scale, rows_grid, blk, 0, st, w, 1.0 / b0, nn, V);
    // The steps run without a host round trip: alpha_j and beta_j stay on the
    // device until the end. A breakdown (beta_j = 0, an invariant subspace)
    // is found afterwards; the steps after it hold non-finite values that no
    // Ritz vector uses.
    double* alpha_d = ab;
    double* beta_d = ab + ncv;
    for (int j = 0; j < ncv; ++j) {
        hipLaunchKernelGGL(kvb::k_spmv, spmv_grid, blk, 0, st, rowptr, col, val, V + size_t(j) * ldv, nn, w);
        // two passes of classical Gram-Schmidt against v_0..v_j; alpha_j is
        // the first pass's coefficient on v_j plus the second's correction
        for (int pass = 0; pass < 2; ++pass) {
            project(V, w, j + 1);
            hipLaunchKernelGGL(kvb::k_project_sum, dim3((j + 64) / 64), dim3(64), 0, st, part, j + 1, nchunk, ldp, h,
                               pass == 0 ? 1 : 0, alpha_d + j);
            hipLaunchKernelGGL(kvb::k_subtract_span, dim3((nn + 63) / 64), dim3(64), 0, st, V, ldv, j + 1, h, nn, w);
        }
        // beta_j = ||w||, v_{j+1} = w / beta_j (V has room for v_ncv)
        project(w, w, 1);
        hipLaunchKernelGGL(kvb::k_scale_by_norm, rows_grid, blk, 0, st, w, part, nchunk, ldp, nn,
                           V + size_t(j + 1) * ldv, beta_d + j);
        KVB_HIP(ctx, hipGetLastError());
    }
    std::vector<double> abh(2 * size_t(ncv));
    KVB_HIP(ctx, hipMemcpyAsync(abh.data(), ab, sizeof(double) * abh.size(), hipMemcpyDeviceToHost, st));
    KVB_HIP(ctx, hipStreamSynchronize(st));
    int m = 0;
    if (kvb_lanczos_prefix(abh.data(), abh.data() + ncv, ncv, &m) != KVB_OK)
        return fail(ctx, KVB_E_INVALID, "non-finite Lanczos coefficient after %d steps: the matrix or the "
                    "start vector holds non-finite values", m);
    std::vector<double> alpha(abh.begin(), abh.begin() + m);
    std::vector<double> beta(abh.begin() + ncv, abh.begin() + ncv + m);
    if (m < ncv) beta[size_t(m) - 1] = 0.0;   // invariant subspace found: the Ritz pairs are exact
    KVB_REQUIRE(ctx, nev <= m, "the Krylov space closed after %d steps, below nev = %d", m, nev);
    // Ritz pairs of T
    std::vector<double> theta, Yt;
    top_eigenpairs(alpha, beta, m, nev, theta, Yt);
    double scale = 0.0;
    for (int i = 0; i < m; ++i)
        scale = std::max(scale, std::fabs(alpha[i]) + (i > 0 ? std::fabs(beta[i - 1]) : 0.0) +
                                    (i + 1 < m ? std::fabs(beta[i]) : 0.0));
    bool converged = true;
    std::vector<double> Ssel(size_t(m) * nev);
    for (int q = 0; q < nev; ++q) {
        evals_host[q] = theta[q];
        const double res = std::fabs(beta[m - 1] * Yt[size_t(q) * m + m - 1]);
        if (resid_host) resid_host[q] = res;
        if (res > tol * scale) converged = false;
        for (int c = 0; c < m; ++c) Ssel[size_t(c) * nev + q] = Yt[size_t(q) * m + c];
    }
    if (evecs) {
        KVB_HIP(ctx, hipMemcpyAsync(S, Ssel.data(), sizeof(double) * Ssel.size(), hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(kvb::k_ritz, dim3(rows_grid.x, (nev + kvb::RITZ_VECS - 1) / kvb::RITZ_VECS), blk, 0, st, V, ldv, m, S, nev, nn, evecs);
        KVB_HIP(ctx, hipGetLastError());
        KVB_HIP(ctx, hipStreamSynchronize(st));
    }
    return converged ? KVB_OK : KVB_W_NOT_CONVERGED;
}

int kvb_kolmogorov_solve(kvb_ctx ctx, const double* evecs, const double* evals_host, int32_t nvec, int32_t skip,
                         const double* P, const double* D, const double* g, int64_t n, double* f, double* g_proj,
                         double* coef_host)
{
    if (!ctx) return KVB_E_INVALID;
    KVB_REQUIRE(ctx, n >= 1 && n < (int64_t(1) << 31), "n must be in [1, 2^31)");
    KVB_REQUIRE(ctx, nvec >= 1 && skip >= 0 && skip < nvec && nvec <= 1024, "need 0 <= skip < nvec <= 1024");
    KVB_REQUIRE(ctx, evals_host != nullptr, "evals_host must be non-null");
    KVB_REQUIRE(ctx, aligned(evecs) && aligned(P) && aligned(D) && aligned(g) && aligned(f),
                "evecs, P, D, g, f must be non-null float64 device pointers");
    KVB_REQUIRE(ctx, g_proj == nullptr || aligned(g_proj), "g_proj must be aligned");
    const int l = nvec - skip;
    for (int j = skip; j < nvec; ++j)
        KVB_REQUIRE(ctx, evals_host[j] != 0.0 && std::isfinite(evals_host[j]),
                    "eigenvalue %d is zero or not finite: skip the null pairs", j);
    const int nn = static_cast<int>(n);
    int rc = ensure_scratch(ctx, round256(size_t(nn) * sizeof(double)) + 3 * round256(size_t(l) * sizeof(double)) + 1024);
    if (rc) return rc;
    Carve cv(ctx->scratch);
    double* part = cv.take<double>(nn);
    double* c = cv.take<double>(l);
    double* cf = cv.take<double>(l);
    double* cg = cv.take<double>(l);
    hipStream_t st = ctx->stream;
    const double* Y = evecs + size_t(skip) * nn;
    const dim3 blk(256), rows_grid(static_cast<unsigned>((n + 255) / 256));
    double* lam = ctx->spec_host;
    double* ch = ctx->spec_host + SPEC_MAX;
    for (int j = 0; j < l; ++j) lam[j] = evals_host[skip + j];
    const RowChunks rk = row_chunks(nn, l);
    double* pt = rk.count > 1 ? part : c;
    hipLaunchKernelGGL((kvb::k_project_chunk<1, true>), dim3((l + kvb::SP_VECS - 1) / kvb::SP_VECS, rk.count), blk, 0,
                       st, Y, l, g, g, P, D, nn, rk.rows, pt);
    hipLaunchKernelGGL(kvb::k_solve_coef, dim3((l + 3) / 4), blk, 0, st, pt, rk.count, l, lam, cf, cg, ch);
    hipLaunchKernelGGL(kvb::k_expand, rows_grid, blk, 0, st, Y, l, cf, cg, P, D, nn, f, g_proj);
    KVB_HIP(ctx, hipGetLastError());
    KVB_HIP(ctx, hipStreamSynchronize(st));
    if (coef_host) {
        // the paper's coefficients g~_j = <phi_j, g>_S with <phi_i, phi_j>_S = delta_ij, phi_j = sqrt(n) S^{-1} y_j
        const double rn = 1.0 / std::sqrt(static_cast<double>(n));
        for (int j = 0; j < l; ++j) coef_host[j] = ch[j] * rn;
    }
    return KVB_OK;
}

int kvb_carre_du_champ(kvb_ctx ctx, const double* evecs, const double* evals_host, int32_t nvec, const double* P,
                       const double* D, const double* u, const double* v, int64_t n, double* grad, double* C)
{
    if (!ctx) return KVB_E_INVALID;
    KVB_REQUIRE(ctx, n >= 1 && n < (int64_t(1) << 31), "n must be in [1, 2^31)");
    KVB_REQUIRE(ctx, nvec >= 1 && nvec <= 1024, "need 1 <= nvec <= 1024");
    KVB_REQUIRE(ctx, C == nullptr || nvec <= kvb::CDC_MAX, "the coefficient tensor needs nvec <= %d", kvb::CDC_MAX);
    KVB_REQUIRE(ctx, evals_host != nullptr, "evals_host must be non-null");
    KVB_REQUIRE(ctx, aligned(evecs) && aligned(P) && aligned(D) && aligned(u) && aligned(v) && aligned(grad),
                "evecs, P, D, u, v, grad must be non-null float64 device pointers");
    KVB_REQUIRE(ctx, C == nullptr || aligned(C), "C must be aligned");
    const int nn = static_cast<int>(n);
    const int npairs = nvec * (nvec + 1) / 2;
    int rc = ensure_scratch(ctx, 4 * round256(size_t(nn) * sizeof(double)) + 6 * round256(size_t(nvec) * sizeof(double)) +
                                     2 * round256(size_t(npairs) * sizeof(int)) + 2048);
    if (rc) return rc;
    Carve cv(ctx->scratch);
    double* part = cv.take<double>(2 * size_t(nn));
    double* t1 = cv.take<double>(nn);
    double* t2 = cv.take<double>(nn);
    double* pq = cv.take<double>(2 * size_t(nvec));
    double* coef = cv.take<double>(4 * size_t(nvec));
    int* pj = cv.take<int>(npairs);
    int* pk = cv.take<int>(npairs);
    hipStream_t st = ctx->stream;
    const dim3 blk(256), rows_grid(static_cast<unsigned>((n + 255) / 256)), coef_grid((nvec + 3) / 4);
    double* lam = ctx->spec_host;
    for (int j = 0; j < nvec; ++j) lam[j] = evals_host[j];
    const RowChunks rk = row_chunks(nn, nvec);
    const dim3 proj_grid((nvec + kvb::SP_VECS - 1) / kvb::SP_VECS, rk.count);
    double* pt = rk.count > 1 ? part : pq;
    hipLaunchKernelGGL((kvb::k_project_chunk<2, true>), proj_grid, blk, 0, st, evecs, nvec, u, v, P, D, nn,
                       rk.rows, pt);
    hipLaunchKernelGGL(kvb::k_cdc_coef, dim3((2 * nvec + 3) / 4), blk, 0, st, pt, rk.count, nvec, lam, coef);
    hipLaunchKernelGGL(kvb::k_cdc_products, rows_grid, blk, 0, st, evecs, nvec, coef, P, D, nn, t1, t2);
    hipLaunchKernelGGL((kvb::k_project_chunk<2, false>), proj_grid, blk, 0, st, evecs, nvec, t1, t2, P, D, nn,
                       rk.rows, pt);
    hipLaunchKernelGGL(kvb::k_cdc_grad_coef, coef_grid, blk, 0, st, pt, rk.count, nvec, lam, coef);
    hipLaunchKernelGGL(kvb::k_expand, rows_grid, blk, 0, st, evecs, nvec, coef, coef, P, D, nn, grad,
                       static_cast<double*>(nullptr));
    KVB_HIP(ctx, hipGetLastError());
    if (C) {
        std::vector<int> hj(npairs), hk(npairs);
        int q = 0;
        for (int j = 0; j < nvec; ++j)
            for (int k = j; k < nvec; ++k) {
                hj[q] = j;
                hk[q] = k;
                ++q;
            }
        KVB_HIP(ctx, hipMemcpyAsync(pj, hj.data(), sizeof(int) * npairs, hipMemcpyHostToDevice, st));
        KVB_HIP(ctx, hipMemcpyAsync(pk, hk.data(), sizeof(int) * npairs, hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(kvb::k_cdc_tensor, dim3(npairs), blk, 0, st, evecs, nvec, P, D, nn, pj, pk, C);
        KVB_HIP(ctx, hipGetLastError());
    }
    KVB_HIP(ctx, hipStreamSynchronize(st));
    return KVB_OK;
}

int kvb_advect(kvb_ctx ctx, const float* X, int64_t n, int32_t m, const double* velocity, const double* grad,
               const double* noise, double dt, double sigma, float* X_out)
{
    if (!ctx) return KVB_E_INVALID;
    KVB_REQUIRE(ctx, n >= 1 && n < (int64_t(1) << 31) && m >= 1 && n * m < (int64_t(1) << 40), "bad n or m");
    KVB_REQUIRE(ctx, std::isfinite(dt) && dt >= 0 && std::isfinite(sigma), "dt must be finite and >= 0, sigma finite");
    KVB_REQUIRE(ctx, aligned(X) && aligned(grad) && aligned(X_out), "X, grad, X_out must be non-null device pointers");
    KVB_REQUIRE(ctx, (velocity == nullptr || aligned(velocity)) && (noise == nullptr || aligned(noise)),
                "velocity and noise must be aligned");
    const int64_t total = n * m;
    hipLaunchKernelGGL(kvb::k_advect, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, ctx->stream, X,
                       static_cast<int>(n), m, velocity, grad, noise, dt, std::sqrt(dt) * sigma, X_out);
    KVB_HIP(ctx, hipGetLastError());
    return KVB_OK;
}

}  // extern "C"
