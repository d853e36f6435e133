"""Edges of the Lanczos sweeps (run on an MI355X): rows that fill no
workgroup, a space as large as the matrix, bases that end inside a group of
four vectors, one and several row chunks, empty rows.

Checked on what defines the result: the Ritz vectors are orthonormal, and the
residual A y - theta y has the reported norm. Twice repeated Gram-Schmidt
leaves an orthogonality error of a few times ncv 2^-53, and each matrix-vector
product here errs by at most (64 + 2) 2^-53 of ||A||; both tolerances allow
a factor 16 for the chain of ncv steps' constants.
"""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nev,ncv", [(2, 1, 2), (33, 5, 33), (257, 4, 70), (1000, 6, 530), (20011, 13, 131)])
def test_eigsh_relation_at_sweep_edges(gpu_lib, n, nev, ncv):
    rng = np.random.default_rng(n)
    A = sp.random(n, n, density=min(1.0, 12 / n), random_state=rng, dtype=np.float64)
    A = (A + A.T + sp.diags(np.linspace(-1, 1, n))).tocsr().astype(np.float32)
    empty = n // 2
    if n > 2:          # a row and column without entries
        keep = sp.diags((np.arange(n) != empty).astype(np.float32))
        A = (keep @ A @ keep).tocsr()
        A.eliminate_zeros()
    A.sort_indices()
    e = gpu_lib.eigsh(torch.from_numpy(A.indptr.astype(np.int64)).cuda(),
                      torch.from_numpy(A.indices.astype(np.int32)).cuda(), torch.from_numpy(A.data).cuda(), nev=nev,
                      ncv=ncv, vectors=True)
    Y, Ad = e.vectors.cpu().numpy(), A.astype(np.float64)
    u = 2.0 ** -53
    norm = abs(Ad).sum(1).max()
    assert np.abs(Y @ Y.T - np.eye(nev)).max() <= 16 * ncv * u * 8
    res = np.linalg.norm(Ad @ Y.T - Y.T * e.values, axis=0)
    assert np.abs(res - e.residuals).max() <= 16 * (ncv + 66) * u * norm * 8
