"""Edges of the tuning sums (run on an MI355X): one block of entries, the block
counts where the grid points are split differently and where the partial sums
are added by one launch, and grids that fill no group of 16 or 64 points.

The reference forms the sums in float64. A term's float32 argument is rounded
three times (quotient, coefficient, product), an error of at most
3 t exp(-t) 2^-24 <= 1.2 2^-24, and its exponential by 2 2^-24; every row holds
the term 1, so k such terms err by at most 3.2 k 2^-24 of the sum. A thread adds
at most 16 terms in float32: 16 2^-24 more.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k,G", [(3, 2, 3), (256, 16, 16), (257, 16, 17), (16384, 16, 63), (16385, 16, 64),
                                   (32768, 16, 65), (32769, 16, 256)])
def test_chi_at_block_and_grid_edges(gpu_lib, n, k, G):
    rng = np.random.default_rng(n)
    idx = rng.integers(0, n, (n, k)).astype(np.int32)
    d2 = np.sort(rng.uniform(0, 4, (n, k)), 1).astype(np.float32)
    d2[:, 0] = 0
    rho = rng.uniform(0.5, 2, n).astype(np.float32)
    lo, hi = 0.05, 3.0
    x = d2.astype(np.float64) / (rho[:, None].astype(np.float64) * rho[idx])
    e = np.exp(np.log(lo) + np.arange(G) * (np.log(hi) - np.log(lo)) / (G - 1))
    chi = np.array([np.exp(-x / v).sum() for v in e])
    dev = [torch.from_numpy(a).cuda() for a in (idx, d2, rho)]
    tol = (3.2 * k + 16) * 2.0 ** -24
    t = gpu_lib.tune_eps(*dev, lo, hi, G)
    np.testing.assert_allclose(t.chi, chi, rtol=tol)
    slope = np.diff(np.log(t.chi)) / np.diff(np.log(e))
    assert t.e_star == pytest.approx(e[int(np.argmax(slope))], rel=1e-13)
    rowptr = torch.arange(n + 1, dtype=torch.int64).cuda() * k
    c = gpu_lib.tune_eps_csr(gpu_lib.CsrPattern(rowptr, dev[0].reshape(-1), dev[1].reshape(-1)), dev[2], lo, hi, G)
    np.testing.assert_allclose(c.chi, chi, rtol=tol)
