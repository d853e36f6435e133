"""Edges of the partitioner's backward kernels (run on an MI355X): batches of
one tile, contractions that do not split evenly over the four wavefronts of a
tile or pass what they load ahead, widths that differ from one matrix of a
launch to the next, padded and unpadded input rows.

The inputs make every step exact, so the gradients are compared bit for bit:
small integer samples and sparse integer weights; one bucket's bias so large
that the softmax is exactly one-hot; neighbour counts and a batch that are
powers of two. Every product and sum is then a small multiple of one power of
two (checked below: it survives the BF16 casts and float32 sums).
"""
import numpy as np
import pytest
import torch

from oracle import learned

pytestmark = pytest.mark.gpu

KS = 4


def sparse(rng, rows, cols, per_row):
    w = np.zeros((rows, cols))
    for r in range(rows):
        at = rng.choice(cols, min(cols, per_row), replace=False)
        w[r, at] = rng.choice([-1.0, 1.0], at.size)
    return w


@pytest.mark.parametrize("B,m,h1,h2,nb", [(32, 32, 32, 32, 32), (64, 7, 96, 32, 160), (512, 64, 32, 96, 1184),
                                          (2048, 33, 64, 160, 96)])
def test_backward_exact_at_tile_edges(gpu_lib, B, m, h1, h2, nb):
    kvb = gpu_lib
    rng = np.random.default_rng(B + m)
    X = rng.integers(-1, 2, (B, m)).astype(np.float64)
    W1, W2, W3 = sparse(rng, h1, m, 3), sparse(rng, h2, h1, 2), rng.integers(-1, 2, (nb, h2)).astype(np.float64)
    b1, b2, b3 = rng.integers(0, 2, h1) * 1.0, rng.integers(0, 2, h2) * 1.0, np.zeros(nb)
    hot = nb // 2
    b3[hot] = 65536.0
    lab = rng.integers(0, nb, (B, KS)).astype(np.int32)

    H1 = np.maximum(X @ W1.T + b1, 0)
    H2 = np.maximum(H1 @ W2.T + b2, 0)
    Z = H2 @ W3.T + b3
    assert (Z[:, hot] - np.delete(Z, hot, 1).max(1) > 2000).all() and np.abs(Z).max() < 2 ** 24
    dZ = np.zeros((B, nb))
    dZ[:, hot] = 1
    np.subtract.at(dZ, (np.arange(B)[:, None], lab), 1 / KS)
    dZ /= B
    dH2 = (dZ @ W3) * (H2 > 0)
    dH1 = (dH2 @ W2) * (H1 > 0)
    for t in (X, H1, H2, dZ, dH2, dH1):
        assert np.array_equal(learned.bf16_round(t.astype(np.float32)), t)
    want = [dH1.T @ X, dH1.sum(0), dH2.T @ H1, dH2.sum(0), dZ.T @ H2, dZ.sum(0)]
    assert max(np.abs(t).max() for t in want) * B * KS < 2 ** 24

    ctx = kvb.Context()
    kvb.part_init(m, h1, h2, nb, 2, ctx=ctx)
    flat = learned.flatten([W1, b1, W2, b2, W3, b3]).astype(np.float32)
    kvb.part_set_params(torch.from_numpy(flat).cuda(), ctx=ctx)
    loss, grads = kvb.mlp_backward(torch.from_numpy(X.astype(np.float32)).cuda(), torch.from_numpy(lab).cuda(),
                                   ctx=ctx)
    assert np.array_equal(grads.cpu().numpy(), learned.flatten(want).astype(np.float32))
    want_loss = (Z[:, hot] - Z[np.arange(B)[:, None], lab].mean(1)).mean()
    assert loss == np.float32(want_loss)
    ctx.close()


@pytest.mark.parametrize("nb,P", [(32, 1), (32, 32), (96, 5), (992, 8), (1024, 4), (1024, 9), (1056, 4)])
def test_routes_follow_the_logits(gpu_lib, nb, P):
    # small integer logits: ties by the dozen in every row, to the smaller bucket
    kvb, B, m = gpu_lib, 67, 8
    rng = np.random.default_rng(nb + P)
    X = torch.from_numpy(rng.integers(-1, 2, (B, m)).astype(np.float32)).cuda()
    params = [sparse(rng, 32, m, 3), rng.integers(0, 2, 32) * 1.0, sparse(rng, 32, 32, 2), rng.integers(0, 2, 32) * 1.0,
              sparse(rng, nb, 32, 2), np.zeros(nb)]
    ctx = kvb.Context()
    kvb.part_init(m, 32, 32, nb, P, ctx=ctx)
    kvb.part_set_params(torch.from_numpy(learned.flatten(params).astype(np.float32)).cuda(), ctx=ctx)
    home, probe = kvb.part_route(X, P, ctx=ctx)
    pad = torch.cat([X, X[:(-B) % 32]])
    Z = kvb.mlp_forward(pad, nb, ctx=ctx).cpu().numpy()[:B]
    want = np.argsort(-Z, axis=1, kind="stable")[:, :P]
    np.testing.assert_array_equal(probe.cpu().numpy(), want)
    np.testing.assert_array_equal(home.cpu().numpy(), want[:, 0])
    ctx.close()


@pytest.mark.parametrize("B,h1,h2,nb", [(32768, 64, 256, 1024), (16960, 256, 96, 512), (8192, 1024, 64, 1024)])
def test_large_forward_exact(gpu_lib, B, h1, h2, nb):
    # small integers: every product and sum is exact in BF16 and float32
    kvb, m = gpu_lib, 17
    rng = np.random.default_rng(nb)
    X = rng.integers(-1, 2, (B, m)).astype(np.float32)
    W1, W2, W3 = (sparse(rng, r, c, 3).astype(np.float32) for r, c in ((h1, m), (h2, h1), (nb, h2)))
    b = [rng.integers(0, 2, r).astype(np.float32) for r in (h1, h2, nb)]
    H = np.maximum(X @ W1.T + b[0], 0)
    H = np.maximum(H @ W2.T + b[1], 0)
    want = H @ W3.T + b[2]
    ctx = kvb.Context()
    kvb.part_init(m, h1, h2, nb, 2, ctx=ctx)
    flat = learned.flatten([W1, b[0], W2, b[1], W3, b[2]]).astype(np.float32)
    kvb.part_set_params(torch.from_numpy(flat).cuda(), ctx=ctx)
    np.testing.assert_array_equal(kvb.mlp_forward(torch.from_numpy(X).cuda(), nb, ctx=ctx).cpu().numpy(), want)
    ctx.close()


@pytest.mark.parametrize("nb,P", [(64, 4), (64, 32), (256, 9), (288, 9)])
def test_routes_at_every_row_width(gpu_lib, nb, P):
    # the largest rows of one and of four logits per lane, and one beyond
    test_routes_follow_the_logits(gpu_lib, nb, P)
