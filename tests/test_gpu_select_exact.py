"""Exactness of the curve-ordered selection where its scores are coarse (run on
an MI355X): BF16 scores of one term per coordinate order close candidates
wrongly, so a row's list may lack true neighbours, and only the certificate and
the exact fallback make the row right.

The samples are tight clusters in a 4-dimensional subspace: inside a cluster
the scores' error exceeds the distances. The float64 oracle is the reference.
"""
import numpy as np
import pytest
import torch

import workloads
from parity import check_knn_rows, knn_reference, say

pytestmark = pytest.mark.gpu


def clusters(n, m, radius, seed):
    rng = np.random.default_rng(seed)
    V, _ = np.linalg.qr(rng.standard_normal((m, 4)))
    centres = 2 * rng.standard_normal((5, 4))
    return ((centres[rng.integers(5, size=n)] + radius * rng.standard_normal((n, 4))) @ V.T).astype(np.float32)


def search(kvb, X, k, margin, split, mode="bf16"):
    """kvb_knn into arrays of -1 / NaN, so that an entry left out is seen."""
    n, m = X.shape
    ctx = kvb.Context()
    ctx.set_option(kvb.OPT_BF16_SPLIT, split)
    Xd = torch.from_numpy(X).cuda()
    idx = torch.full((n, k), -1, dtype=torch.int32, device="cuda")
    d2 = torch.full((n, k), float("nan"), device="cuda")
    ctx.check(ctx.lib.kvb_knn(ctx.h, kvb._ptr(Xd), n, m, k, kvb.MODES[mode], margin, kvb._ptr(idx), kvb._ptr(d2), None))
    fallback = kvb.knn_fallback_rows(ctx)
    ctx.close()
    say(f"[select-exact] n={n} m={m} k={k} margin={margin} {mode} split={split}: fallback rows {fallback}")
    return idx.cpu().numpy(), d2.cpu().numpy()


@pytest.mark.parametrize("m", [96, 128])
def test_rows_are_complete(gpu_lib, m):
    """Without a margin a list short of its keys may be short of the row's k - 1
    neighbours: such a row goes to the exact fallback, with every entry written."""
    gi, gd = search(gpu_lib, clusters(12000, m, 0.02, m), 64, 0, 1)
    assert (gi >= 0).all() and not np.isnan(gd).any()
    assert (np.diff(np.sort(gi, axis=1), axis=1) > 0).all()


def check(kvb, X, k, margin, split, mode="bf16", nrows=300):
    gi, gd = search(kvb, X, k, margin, split, mode)
    rows = np.random.default_rng(k).choice(len(X), nrows, replace=False)
    ri, rd = knn_reference(X, k, rows)
    check_knn_rows(gi[rows], gd[rows], ri, rd, k, rows)


@pytest.mark.parametrize("margin", [0, 8, 32])
@pytest.mark.parametrize("m", [96, 128])
def test_coarse_scores(gpu_lib, m, margin):
    for radius in (0.005, 0.02):
        check(gpu_lib, clusters(12000, m, radius, m), 64, margin, 1)
    check(gpu_lib, workloads.gaussian_mixture(16384, seed=m, m=m), 64, margin, 1)
    check(gpu_lib, workloads.sphere3_lifted(20000, seed=m, m=m), 16, margin, 1, nrows=150)
    check(gpu_lib, clusters(12000, 84, 0.02, m), 64, margin, 6)   # 6 m + 3 terms of at most 512


# k and margin on every kind of list: cut at 128 keys, sorted at 128, cut at 256, sorted at 256
LISTS = [(40, 0), (64, 32), (65, 32), (128, 0), (97, 32), (160, 32), (161, 32), (224, 32)]


@pytest.mark.parametrize("m,mode", [(16, "f32"), (16, "bf16"), (64, "bf16"), (100, "f32")])
def test_more_tiles_than_notes(gpu_lib, m, mode):
    # no tile of the unstructured samples can be skipped (some 700 tiles within reach of
    # every query), those of a far cluster can
    X = workloads.gaussian_iid(25000, m, seed=m)
    X[::10] = X[::10] * 0.1 + 40
    for k, margin in LISTS:
        check(gpu_lib, X, k, margin, 3, mode, nrows=500)


@pytest.mark.parametrize("n,m,mode", [(70001, 12, "f32"), (70001, 16, "bf16"), (70001, 31, "f32"),   # short contractions
                                      (25001, 64, "bf16"), (25001, 100, "f32"), (17000, 160, "bf16")])
def test_every_tile_within_reach(gpu_lib, n, m, mode):
    # the query tiles are handed over from the walk to the scans of every tile
    X = workloads.gaussian_iid(n, m, seed=m)
    for k, margin in ((9, 0), (40, 32), (97, 31), (224, 32)):
        check(gpu_lib, X, k, margin, 3, mode, nrows=200)


def test_more_tiles_than_notes_coarse(gpu_lib):
    for margin in (0, 32):
        check(gpu_lib, workloads.gaussian_iid(25000, 100, seed=3), 40, margin, 1, nrows=500)


def test_every_tile_within_reach_coarse(gpu_lib):
    # short contractions of one term: the scan skips tiles by true distances
    X = workloads.gaussian_iid(70001, 40, seed=3)
    X[::2] *= 0.5
    check(gpu_lib, X, 40, 32, 1, nrows=200)


@pytest.mark.parametrize("mode", ["f32", "bf16"])
@pytest.mark.parametrize("k,margin", [(40, 0), (64, 32), (96, 32), (128, 32), (224, 32)])
def test_more_tiles_than_notes_equal_scores(gpu_lib, k, margin, mode):
    # corners of a 12-cube, six or so samples at each: 70 at distance 1, 400 at sqrt 2
    X = np.random.default_rng(k).integers(0, 2, (25000, 12)).astype(np.float32)
    check(gpu_lib, X, k, margin, 3, mode, nrows=500)


@pytest.mark.parametrize("n,m,mode,every", [(25001, 64, "bf16", True),    # every tile scored by the workgroup scan
                                            (70001, 12, "f32", False),    # short contractions: tiles out of reach left out
                                            (25000, 12, "f32", False)])   # the walk beyond its notes
def test_pairs_count_once(gpu_lib, n, m, mode, every):
    ctx = gpu_lib.Context()
    gpu_lib.knn(torch.from_numpy(workloads.gaussian_iid(n, m, seed=m)).cuda(), 64, mode, 32, ctx=ctx)
    pairs = gpu_lib.knn_pairs(ctx)
    ctx.close()
    assert pairs == float(n) * n if every else 0.5 * n * n < pairs <= float(n) * n
