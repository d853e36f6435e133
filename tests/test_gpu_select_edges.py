"""Edges of the curve-ordered selection and of its preparation (run on an
MI355X): sample counts around the tiles, every contraction length on both sides
of the kernel's two forms, list lengths on both sides of the scores kept per
lane and of the list capacities, lists that overflow (exact duplicates beyond
the capacity), and outlying samples whose tiles note more tiles than a
wavefront remembers.

The float64 oracle is the reference; sets and distances are compared by the
rules of parity.py (exact sets where the gap at the k-th neighbour is clear).
"""
import numpy as np
import pytest
import torch

import oracle
import workloads
from parity import check_knn_rows, knn_reference, say

pytestmark = pytest.mark.gpu


def run(kvb, X, k, margin, mode):
    idx, d2, _ = kvb.knn(torch.from_numpy(np.ascontiguousarray(X)).cuda(), k, mode, margin)
    return idx.cpu().numpy(), d2.cpu().numpy()


def check(kvb, X, k, margin, mode):
    say(f"[select-edges] n={len(X)} m={X.shape[1]} k={k} margin={margin} mode={mode}")
    gi, gd = run(kvb, X, k, margin, mode)
    ri, rd = knn_reference(X, k)
    check_knn_rows(gi, gd, ri, rd, k, np.arange(len(X)))


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 96, 97, 129, 257, 2049])
def test_sample_counts(gpu_lib, n):
    for m, mode in ((16, "f32"), (70, "bf16")):
        check(gpu_lib, workloads.gaussian_iid(n, m, seed=n), min(n, 20), 12, mode)


@pytest.mark.parametrize("mode,m", [("f32", m) for m in (9, 12, 15, 31, 32, 47, 63, 64, 95, 127, 128, 191, 255)] +
                         [("bf16", m) for m in (9, 15, 25, 26, 31, 36, 42, 52, 68, 84, 105, 132, 169)])
def test_contraction_lengths(gpu_lib, mode, m):
    check(gpu_lib, workloads.gaussian_mixture(900, seed=m, m=m), 40, 32, mode)


@pytest.mark.parametrize("m", [28, 40, 48, 52, 60, 72, 96, 100, 124, 144, 192, 196, 252])
def test_recomputed_row_lengths(gpu_lib, m):
    # every number of float4 pieces per lane, whole and partial
    check(gpu_lib, workloads.gaussian_mixture(700, seed=m, m=m), 30, 67, "f32")


@pytest.mark.parametrize("k,margin", [(64, 32), (65, 32), (96, 32), (97, 32), (160, 32), (193, 32), (224, 32),
                                      (256, 0)])
def test_list_lengths(gpu_lib, k, margin):
    for m, mode in ((16, "f32"), (64, "bf16")):
        check(gpu_lib, workloads.nonlinear5(3000, seed=k)[:, 64 - m:], k, margin, mode)


@pytest.mark.parametrize("m,mode", [(12, "f32"), (64, "bf16"), (130, "f32")])
def test_duplicates_beyond_the_list(gpu_lib, m, mode):
    # 300 copies of each of 9 lattice points: hundreds of equal scores per list
    base = workloads.cubic_lattice(3)[::3].astype(np.float32)
    X = np.zeros((2700, m), dtype=np.float32)
    X[:, :3] = np.repeat(base, 300, axis=0)[np.random.default_rng(m).permutation(2700)]
    gi, _ = run(gpu_lib, X, 50, 20, mode)
    ri, _ = oracle.knn(X, 50)
    np.testing.assert_array_equal(gi, ri)


@pytest.mark.parametrize("m,mode", [(16, "f32"), (64, "bf16")])
def test_outlying_samples(gpu_lib, m, mode):
    n = 20000
    rng = np.random.default_rng(m)
    X = workloads.gaussian_mixture(n, seed=5, m=m)
    far = rng.choice(n, 200, replace=False)
    X[far] *= rng.uniform(3, 40, (200, 1)).astype(np.float32)
    gi, gd = run(gpu_lib, X, 64, 32, mode)
    rows = np.concatenate([far, rng.choice(n, 300, replace=False)])
    ri, rd = knn_reference(X, 64, rows)
    check_knn_rows(gi[rows], gd[rows], ri, rd, 64, rows)
