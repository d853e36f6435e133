"""Edges of the direct-difference k-NN of few coordinates (run on an MI355X):
sample counts at the edges of its tiles, superblocks and rows per wavefront,
list lengths on both sides of the capacities, every number of coordinates,
samples that repeat beyond a list, and the count of scored pairs.

The float64 oracle is the reference; sets and distances are compared by the
rules of parity.py (exact sets where the gap at the k-th neighbour is clear).
"""
import numpy as np
import pytest
import torch

import oracle
import workloads
from parity import check_knn_rows, say

pytestmark = pytest.mark.gpu


def check(kvb, X, k, margin, ctx=None):
    say(f"[direct-edges] n={len(X)} m={X.shape[1]} k={k} margin={margin}")
    idx, d2, _ = kvb.knn(torch.from_numpy(np.ascontiguousarray(X)).cuda(), k, "f32", margin, ctx)
    rows = np.unique(np.linspace(0, len(X) - 1, min(len(X), 600)).astype(np.int64))
    ri, rd = oracle.knn_sampled(X, min(k + 1, len(X)), rows)
    check_knn_rows(idx.cpu().numpy()[rows], d2.cpu().numpy()[rows], ri, rd, k, rows)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 257, 448, 1024, 1025, 4097, 32768, 32769, 65541])
def test_sample_counts(gpu_lib, n):
    check(gpu_lib, workloads.gaussian_iid(n, 3, seed=n), min(n, 20), 8)


@pytest.mark.parametrize("k,margin", [(1, 0), (2, 0), (56, 8), (57, 8), (64, 0), (65, 0), (120, 8), (121, 8), (248, 8),
                                      (256, 0)])
def test_list_lengths(gpu_lib, k, margin):
    for n in (300, 3001, 33000):
        check(gpu_lib, workloads.torus(n, seed=k), k, margin)


@pytest.mark.parametrize("m", range(1, 9))
def test_coordinates(gpu_lib, m):
    for n in (900, 33001):
        check(gpu_lib, workloads.gaussian_iid(n, m, seed=m), 33, 8)


@pytest.mark.parametrize("copies,k", [(100, 20), (300, 90), (700, 20), (700, 200)])
def test_duplicates_beyond_the_list(gpu_lib, copies, k):
    # equal scores by the hundred: ties at the k-th neighbour go to the smaller index
    rng = np.random.default_rng(copies)
    X = np.repeat(rng.integers(-2, 3, (9, 3)).astype(np.float32), copies, axis=0)[rng.permutation(9 * copies)]
    idx, d2, _ = gpu_lib.knn(torch.from_numpy(X).cuda(), k, "f32", 8)
    ri, rd = oracle.knn(X, k)
    np.testing.assert_array_equal(idx.cpu().numpy(), ri)
    np.testing.assert_array_equal(d2.cpu().numpy(), rd.astype(np.float32))


def test_outlying_samples(gpu_lib):
    # two far clusters and single samples at many scales: boxes that span whole regions
    rng = np.random.default_rng(5)
    X = rng.normal(size=(6000, 3)).astype(np.float32)
    X[3000:] += 1e4
    X[::97] *= np.float32(10.0) ** rng.integers(-6, 7, (len(X[::97]), 1)).astype(np.float32)
    check(gpu_lib, X, 50, 8)


@pytest.mark.parametrize("n", [1, 64, 255, 256])
def test_every_pair_counted(gpu_lib, n):
    # up to four tiles every wavefront scores all of them
    ctx = gpu_lib.Context()
    check(gpu_lib, workloads.gaussian_iid(n, 3, seed=n), 1, 0, ctx)
    assert gpu_lib.knn_pairs(ctx) == n * n


@pytest.mark.parametrize("m", [5, 6, 8])
@pytest.mark.parametrize("k,margin", [(8, 24), (24, 9), (56, 8), (64, 0), (88, 8), (97, 31), (192, 32), (225, 0), (256, 0)])
def test_list_lengths_by_coordinates(gpu_lib, m, k, margin):
    # buffers cut after 32 or 64 further keys, and filled ones, on both sides of each length
    for n in (300, 3001):
        check(gpu_lib, workloads.gaussian_iid(n, m, seed=k), k, margin)


@pytest.mark.parametrize("copies,k", [(100, 20), (300, 90), (700, 20), (700, 200)])
def test_duplicates_in_eight_coordinates(gpu_lib, copies, k):
    rng = np.random.default_rng(copies)
    X = np.repeat(rng.integers(-2, 3, (9, 8)).astype(np.float32), copies, axis=0)[rng.permutation(9 * copies)]
    idx, d2, _ = gpu_lib.knn(torch.from_numpy(X).cuda(), k, "f32", 8)
    ri, rd = oracle.knn(X, k)
    np.testing.assert_array_equal(idx.cpu().numpy(), ri)
    np.testing.assert_array_equal(d2.cpu().numpy(), rd.astype(np.float32))


@pytest.mark.parametrize("n", [262144, 262145, 262146, 262147])
def test_rows_per_wavefront_in_six_coordinates(gpu_lib, n):
    # two rows up to 262144 samples, then three; the last wavefront has 2, 2, 3 and 1
    check(gpu_lib, workloads.gaussian_iid(n, 6, seed=1), 30, 32)
