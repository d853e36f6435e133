"""Edges of the spectral projections' split over basis vectors and row chunks
(run on an MI355X): one and several chunks, a last chunk and a last vector
group that are not full, more vectors than rows allow chunks, against float64
torch on the same inputs.

Tolerance: every output is a short chain of float64 sums of n terms (the
projection, the expansion over nvec vectors, their products); each sum errs by
at most (n + 64) 2^-53 of its absolute terms, and the widest chain here is
three sums long, so 8 (n + nvec) 2^-53 of the same expression in absolute
values bounds it.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nvec", [(37, 5), (511, 1), (512, 4), (1025, 7), (700, 700), (33000, 36), (70001, 9)])
def test_spectral_calls_at_chunk_edges(gpu_lib, n, nvec):
    kvb = gpu_lib
    g = torch.Generator(device="cuda").manual_seed(n + nvec)

    def rnd(*shape):
        return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)

    Y = (rnd(nvec, n) - 0.5) / n ** 0.5
    P, D = 0.5 + rnd(n), 1 + rnd(n)
    u, v, rhs = rnd(n) - 0.5, rnd(n) - 0.5, rnd(n) - 0.5
    lam = -1.0 - np.arange(nvec, dtype=np.float64)
    tl = torch.from_numpy(lam).cuda()
    e = kvb.Eigs(lam, np.zeros(nvec), Y, True)
    S = P * D.sqrt()

    def both(fn):
        """fn on the values and on their absolute values (the error's scale)"""
        a = fn(Y, S, tl, u, v, rhs, 1)
        b = fn(Y.abs(), S, tl.abs(), u.abs(), v.abs(), rhs.abs(), 0)
        return a, b

    def solve(Y, S, lam, u, v, rhs, signed):
        c = (Y * (S * rhs)).sum(1)
        return ((c / lam)[:, None] * Y).sum(0) / S, (c[:, None] * Y).sum(0) / S

    def cdc(Y, S, lam, u, v, rhs, signed):
        p, q = (Y * (S * u)).sum(1), (Y * (S * v)).sum(1)
        at = lambda w: (w[:, None] * Y).sum(0) / S  # noqa: E731
        U, V, LU, LV = at(p), at(q), at(lam * p), at(lam * q)
        a, b = (Y * (S * U * V)).sum(1), (Y * (S * (LU * V + U * LV))).sum(1)
        return at(0.5 * (lam * a - b if signed else lam * a + b))

    tol = 8 * (n + nvec) * 2.0 ** -53
    f, gl, coef = kvb.kolmogorov_solve(e, P, D, rhs, skip=0)
    (rf, rg), (sf, sg) = both(solve)
    assert bool(((f - rf).abs() <= tol * sf).all()) and bool(((gl - rg).abs() <= tol * sg).all())
    c = (Y * (S * rhs)).sum(1) / n ** 0.5
    assert bool((torch.from_numpy(coef).cuda() - c).abs().max() <= tol * (Y * (S * rhs)).abs().sum(1).max())
    grad, _ = kvb.carre_du_champ(e, P, D, u, v)
    r, s = both(cdc)
    assert bool(((grad - r).abs() <= tol * s).all())


def test_solve_at_the_largest_sample_count(gpu_lib):
    """The last row chunk ends beyond 2^31 rows: its rows count, and no row is read
    past the end. One constant eigenvector and unit weights, 17 GB an array; every
    sum is a small whole number."""
    kvb = gpu_lib
    n = 2 ** 31 - 32
    if torch.cuda.mem_get_info()[0] < 100e9:
        pytest.skip("needs 70 GB of device memory")
    one = torch.ones(n, device="cuda", dtype=torch.float64)
    g = torch.zeros(n, device="cuda", dtype=torch.float64)
    rows = [0, n // 2, n - 40, n - 1]
    for r, v in zip(rows, (7.0, 4.0, 5.0, 3.0)):
        g[r] = v
    f = torch.empty(n, device="cuda", dtype=torch.float64)
    lam, coef = np.array([-2.0]), np.zeros(1)
    ctx = kvb.Context()
    at = [kvb._ptr(t) for t in (one, g, f)]
    ctx.check(ctx.lib.kvb_kolmogorov_solve(ctx.h, at[0], lam.ctypes.data, 1, 0, at[0], at[0], at[1], n, at[2], None,
                                           coef.ctypes.data))
    assert coef[0] == 19.0 * (1.0 / np.sqrt(float(n)))
    assert [float(f[r]) for r in rows] == [-9.5] * 4
    ctx.close()
    del one, g, f
    torch.cuda.empty_cache()
