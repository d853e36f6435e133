"""Cases that measure the framework through its public entry points.

Each case is one call (or one short chain of calls) that a program using the
library makes: whole kernel-matrix builds over the range of sizes, dimensions,
modes and patterns, the learned search, the partitioner's gradients, the
eigensolver and the spectral solves. ``exact`` states the same results in
float64 with plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2104_15124_amd import kvb

G, K0, E_MIN, E_MAX, BETA = 64, 8, 1e-3, 1e1, -0.5
OUT_KINDS = {"markov": kvb.OUT_MARKOV, "generator": kvb.OUT_GENERATOR, "symmetric": kvb.OUT_SYMMETRIC}
EXACT_ROWS = 105_000          # largest sample count whose k-NN is searched by brute force in float64


def _build(name, data, n, m, d, k, mode="f32", pattern="knn", delta=0.0, out="markov", api="build"):
    c = dict(name=name, kind="build", data=data, n=n, m=m, d=d, k=k, mode=mode, pattern=pattern, delta=delta,
             out=out, api=api)
    return c if name else {key: v for key, v in c.items() if key != "name"}


def listed():
    return [
        # a first try at a prompt: the small unit sphere, where launches and latency count
        _build("build_sphere_n2000", "sphere", 2000, 3, 2, 32),
        # an ordinary data set of a physics problem: a torus in R^3
        _build("build_torus_n100k", "torus", 100_000, 3, 2, 64),
        # the matrix of an eigenproblem: symmetric pattern and conjugate, small entries dropped, paper-sized
        _build("build_sym_gauss_n25k", "gauss4", 25_000, 4, 4, 25, pattern="union", delta=1e-2, out="symmetric"),
        # the largest data set of few coordinates: a mixture on a linear subspace
        _build("build_mixture_n8m", "mixture", 8_000_000, 16, 4, 64),
        # the same kind of data at a size that fits no tile, in the BF16 form
        _build("build_mixture_bf16_n1m", "mixture", 1_000_003, 16, 4, 64, mode="bf16"),
        # a curved manifold with noise in many coordinates, in the BF16 form
        _build("build_manifold5_bf16_n1m", "manifold5", 1_000_000, 64, 5, 64, mode="bf16"),
        # long rows and many neighbours at the largest size of that kind
        _build("build_sphere3_bf16_n4m", "sphere3", 4_000_000, 128, 3, 128, mode="bf16"),
        # long feature vectors in full precision, odd sizes, through the separate calls
        _build("stages_wide_n30k", "manifold5", 30_011, 200, 5, 32, api="stages"),
        # approximate search with a partitioner that is already there
        dict(name="learned_sphere3_n1m", kind="learned", data="sphere3", n=1_000_000, m=128, k=128, buckets=1024,
             probe=4),
        # one training batch of the partitioner: loss and gradients
        dict(name="partitioner_grad_b512", kind="grad", batch=512, m=128, h1=256, h2=256, buckets=1024, ks=128),
        # the spectrum of an operator on an ordinary data set, with the pairs the density evolution asks for
        dict(name="eigsh_n100k", kind="eigsh", rows=316, cols=316, nev=36, ncv=400),
        # one solve and one gradient on that spectrum
        dict(name="spectral_n100k", kind="spectral", n=100_000, nvec=36, coords=3),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["low", "low", "low", "mid", "mid", "mid", "high", "high", "wide", "learned", "grad", "eigsh",
                         "spectral"])
    if family == "low":
        data, m, d = rng.choice([("sphere", 3, 2), ("torus", 3, 2), ("gauss4", 4, 4)])
        union = rng.random() < 0.4
        return _build("", data, _logint(rng, 1000, 1_000_000), m, d, rng.randint(12, 64 if union else 128),
                      pattern="union" if union else "knn", delta=rng.choice([0.0, 0.0, 1e-2]),
                      out=rng.choice(["markov", "generator", "symmetric"]))
    if family == "mid":
        return _build("", "mixture", _logint(rng, 2000, 3_000_000), rng.randint(9, 39), 4, rng.randint(16, 96),
                      mode=rng.choice(["f32", "bf16"]), api=rng.choice(["build", "build", "stages"]))
    if family == "high":
        if rng.random() < 0.5:
            return _build("", "manifold5", _logint(rng, 2000, 400_000), rng.randint(32, 96), 5, rng.randint(16, 64),
                          mode=rng.choice(["f32", "bf16"]))
        return _build("", "sphere3", _logint(rng, 2000, 800_000), rng.randint(40, 169), 3, rng.randint(16, 128),
                      mode=rng.choice(["f32", "bf16"]))
    if family == "wide":
        return _build("", "manifold5", _logint(rng, 2000, 50_000), rng.randint(97, 255), 5, rng.randint(16, 64),
                      api="stages")
    if family == "learned":
        return dict(kind="learned", data="sphere3", n=_logint(rng, 50_000, 1_000_000), m=rng.randint(12, 128),
                    k=rng.randint(16, 128), buckets=rng.choice([128, 256, 512, 1024]), probe=rng.randint(1, 6))
    if family == "grad":
        return dict(kind="grad", batch=32 * rng.randint(1, 64), m=rng.randint(8, 128), h1=32 * rng.randint(2, 8),
                    h2=32 * rng.randint(2, 8), buckets=32 * rng.randint(4, 32), ks=rng.randint(16, 128))
    if family == "eigsh":
        return dict(kind="eigsh", rows=_logint(rng, 40, 400), cols=_logint(rng, 40, 400), nev=rng.randint(6, 24),
                    ncv=rng.randint(60, 300))
    return dict(kind="spectral", n=_logint(rng, 1000, 500_000), nvec=rng.randint(6, 48), coords=rng.randint(2, 4))


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _samples(data, n, m, seed):
    """Seeded samples [n, m] float32: the distributions of this repository's workloads."""
    g = _gen(seed)

    def randn(*shape):
        return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)

    def rand(*shape):
        return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)

    if data == "sphere":
        x = randn(n, 3)
        return x / x.norm(dim=1, keepdim=True)
    if data == "torus":           # tube angle von Mises(0, 1), azimuth uniform, radii 1 and 2
        t = torch.linspace(-math.pi, math.pi, 8193, dtype=torch.float64, device="cuda")
        pdf = torch.exp(torch.cos(t))
        cdf = torch.cat([torch.zeros(1, dtype=torch.float64, device="cuda"), torch.cumsum(pdf[1:] + pdf[:-1], 0)])
        cdf = cdf / cdf[-1]
        u, phi = rand(n), 2 * math.pi * rand(n)
        i = torch.searchsorted(cdf, u).clamp(1, 8192)
        th = t[i - 1] + (t[i] - t[i - 1]) * (u - cdf[i - 1]) / (cdf[i] - cdf[i - 1])
        r = 2 + torch.cos(th)
        return torch.stack([r * torch.cos(phi), r * torch.sin(phi), torch.sin(th)], 1).float().contiguous()
    if data == "gauss4":          # the paper's 4-D Gaussian
        return randn(n, 4) * torch.tensor([2.0, 2.0, 3.0, 3.0], device="cuda") ** 0.25
    if data == "mixture":         # three unit Gaussians, means 3 apart, on a 4-dimensional subspace
        V = torch.linalg.qr(randn(m, 4).cpu())[0].cuda()
        mu = torch.zeros(3, 4, device="cuda")
        for a in range(3):
            mu[a, a] = 3 / math.sqrt(2)
        u = torch.rand(n, generator=g, device="cuda")
        z = mu[(u > 0.5).long() + (u > 0.8).long()] + randn(n, 4)
        return (z @ V.T).contiguous()
    if data == "manifold5":       # [Q z, sin(W z)] + noise, z in R^5
        h = m // 2
        Q = torch.linalg.qr(randn(h, 5).cpu())[0].cuda()
        W = 0.5 * randn(m - h, 5)
        x = torch.empty(n, m, device="cuda")
        z = randn(n, 5)
        x[:, :h] = z @ Q.T
        x[:, h:] = torch.sin(z @ W.T)
        x += 1e-3 * randn(n, m)
        return x
    U = torch.linalg.qr(randn(m, 4).cpu())[0].cuda()          # uniform S^3 lifted to R^m
    z = randn(n, 4)
    return ((z / z.norm(dim=1, keepdim=True)) @ U.T).contiguous()


def _network(c, seed):
    """He-normal weights in the partitioner's order W1, b1, W2, b2, W3, b3."""
    g = _gen(seed + 7919)
    m, h1, h2, nb = c["m"], c["h1"], c["h2"], c["buckets"]

    def layer(o, i):
        w = torch.randn(o, i, generator=g, device="cuda") * math.sqrt(2 / i)
        return w, 0.05 * torch.randn(o, generator=g, device="cuda")

    return [*layer(h1, m), *layer(h2, h1), *layer(nb, h2)]


def _nearest_centre_network(X, buckets, seed):
    """Weights whose logits are 2 c_b . x - |c_b|^2 for `buckets` samples c_b: a trained-like routing."""
    m = X.shape[1]
    h = (2 * m + 31) // 32 * 32
    at = torch.randperm(X.shape[0], generator=torch.Generator().manual_seed(seed))[:buckets]
    C = X[at.cuda()]
    W1 = torch.zeros(h, m, device="cuda")
    W1[:m] = torch.eye(m, device="cuda")
    W1[m:2 * m] = -torch.eye(m, device="cuda")
    W2 = torch.eye(h, device="cuda")
    W3 = torch.zeros(buckets, h, device="cuda")
    W3[:, :m] = 2 * C
    W3[:, m:2 * m] = -2 * C
    zero = torch.zeros(h, device="cuda")
    return h, torch.cat([t.reshape(-1) for t in (W1, zero, W2, zero, W3, -(C * C).sum(1))])


def _operator(rows, cols, seed):
    """A symmetric CSR operator D^-1/2 K D^-1/2 - I: Gaussian weights between the jittered sites of a periodic
    rows x cols grid of uneven density, about 69 neighbours a site, the sites in random order."""
    g = _gen(seed)
    n = rows * cols
    i = torch.arange(n, device="cuda")
    a, b = i // cols, i % cols
    jit = 0.6 * (torch.rand(n, 2, generator=g, device="cuda", dtype=torch.float64) - 0.5)
    w = 1 + 0.4 * torch.sin(2 * math.pi * a / rows + 0.3) + 0.3 * torch.cos(2 * math.pi * b / cols + 1.1)
    R, C, V = [], [], []
    for da in range(-4, 5):
        for db in range(-4, 5):
            if da * da + db * db <= 22:
                j = ((a + da) % rows) * cols + (b + db) % cols
                dx, dy = da + jit[j, 0] - jit[i, 0], db + jit[j, 1] - jit[i, 1]
                R.append(i)
                C.append(j)
                V.append(torch.exp(-(dx * dx + dy * dy) / 4) * (w * w[j]))
    order = torch.randperm(n, generator=g, device="cuda")
    R, C, V = torch.cat(R), torch.cat(C), torch.cat(V)
    q = torch.zeros(n, dtype=torch.float64, device="cuda")
    for s in range(0, R.numel(), n):          # one neighbour offset at a time: the same sums in every run
        q += V[s:s + n]
    V = V / (q[R] * q[C]).sqrt() - (R == C).double()
    at = torch.argsort(order[R] * n + order[C])
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(order[R], minlength=n), 0)
    return rowptr, order[C][at].int().contiguous(), V[at].float().contiguous()


def _spectrum(n, nvec, coords, seed):
    """Unit vectors like an operator's leading eigenvectors (smooth functions of the samples), the null one first."""
    g = _gen(seed)
    th = 2 * math.pi * torch.rand(n, 2, generator=g, device="cuda", dtype=torch.float64)
    P = 0.1 * torch.exp(0.3 * torch.cos(th[:, 0]))
    D = 60 * torch.exp(0.2 * torch.sin(th[:, 1]))
    S = P * D.sqrt()
    F = [torch.ones(n, dtype=torch.float64, device="cuda")]
    j = 1
    while len(F) < nvec:
        for p in range(j + 1):
            F += [torch.cos(p * th[:, 0] + (j - p) * th[:, 1]), torch.sin(p * th[:, 0] + (j - p) * th[:, 1])]
        j += 1
    Y = torch.stack(F[:nvec], 0) * S
    for _ in range(2):
        L = torch.linalg.cholesky((Y @ Y.T).cpu())
        Y = torch.linalg.solve_triangular(L, torch.eye(nvec, dtype=torch.float64), upper=False).cuda() @ Y
    lam = np.array([-0.17 * i for i in range(nvec)])
    X = torch.stack([torch.sin(th[:, s % 2] * (1 + s // 2) + s) for s in range(coords)])
    return Y.contiguous(), lam, P, D, X, torch.cos(th[:, 0]) + 0.3 * torch.sin(2 * th[:, 1])


def _varying(c):
    """Whether the number of stored entries depends on the samples."""
    return c["pattern"] != "knn" or c["delta"] > 0


def _arrays(c):
    """The arrays of a matrix whose entries vary in number, kept by the caller at their capacity."""
    n, k = c["n"], c["k"]
    cap = n * (2 * k - 1) if c["pattern"] == "union" else n * k

    def zeros(*shape, dtype=torch.float32):
        return torch.zeros(*shape, dtype=dtype, device="cuda")

    return kvb.KernelMatrix(idx=zeros(n, k, dtype=torch.int32), d2=zeros(n, k), flags=zeros(n, dtype=torch.int32),
                            b=zeros(n), tune_a=None, rho=zeros(n), psi=zeros(n), scale_b=None, tune_b=None,
                            rowptr=zeros(n + 1, dtype=torch.int64), col=zeros(cap, dtype=torch.int32),
                            val=zeros(cap), P=zeros(n, dtype=torch.float64), D=zeros(n, dtype=torch.float64))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "build":
        X = _samples(case["data"], case["n"], case["m"], seed)
        return {"c": case, "X": X, "out": _arrays(case) if _varying(case) else None}
    if kind == "learned":
        X = _samples(case["data"], case["n"], case["m"], seed)
        h, params = _nearest_centre_network(X, case["buckets"], seed)
        ctx = kvb.Context()
        kvb.part_init(case["m"], h, h, case["buckets"], case["probe"], seed, ctx=ctx)
        kvb.part_set_params(params, ctx=ctx)
        return {"c": case, "X": X, "ctx": ctx}
    if kind == "grad":
        g = _gen(seed)
        X = torch.randn(case["batch"], case["m"], generator=g, device="cuda")
        home = torch.randint(case["buckets"], (case["batch"], 1), generator=g, device="cuda")
        near = (home + torch.randint(4, (case["batch"], case["ks"]), generator=g, device="cuda")) % case["buckets"]
        ctx = kvb.Context()
        kvb.part_init(case["m"], case["h1"], case["h2"], case["buckets"], 4, seed, ctx=ctx)
        kvb.part_set_params(torch.cat([t.reshape(-1) for t in _network(case, seed)]), ctx=ctx)
        return {"c": case, "X": X, "near": near.int().contiguous(), "ctx": ctx}
    if kind == "eigsh":
        return {"c": case, "csr": _operator(case["rows"], case["cols"], seed)}
    Y, lam, P, D, X, g = _spectrum(case["n"], case["nvec"], case["coords"], seed)
    return {"c": case, "eigs": kvb.Eigs(lam, np.zeros_like(lam), Y, True), "P": P, "D": D, "X": X, "g": g}


# ------------------------------------------------------------------ one pass
def run(state):
    c = state["c"]
    if c["kind"] == "build":
        args = (state["X"], c["k"], K0, float(c["d"]), -c["d"] / 4, BETA, E_MIN, E_MAX, G)
        if c["api"] == "stages":
            km = kvb.build_kernel_matrix(*args, mode=c["mode"], out_kind=OUT_KINDS[c["out"]])
        elif _varying(c):      # into the caller's arrays, then the wait for the tuning
            km = kvb.build(*args, mode=c["mode"], out_kind=OUT_KINDS[c["out"]], pattern=c["pattern"],
                           delta=c["delta"], out=state["out"], sync=False)
            km.tune_a, km.scale_b, km.tune_b, _ = kvb.build_info(G)
        else:
            km = kvb.build(*args, mode=c["mode"], out_kind=OUT_KINDS[c["out"]], pattern=c["pattern"],
                           delta=c["delta"])
        return {"idx": km.idx, "d2": km.d2, "flags": km.flags, "b": km.b, "chi_a": km.tune_a.chi,
                "e_a": km.tune_a.e_star, "dim_a": km.tune_a.dim, "rho": km.rho, "psi": km.psi,
                "scale_b": km.scale_b, "chi_b": km.tune_b.chi, "e_b": km.tune_b.e_star, "dim_b": km.tune_b.dim,
                "rowptr": km.rowptr, "col": km.col, "val": km.val, "P": km.P, "D": km.D}
    if c["kind"] == "learned":
        idx, d2, flags = kvb.knn(state["X"], c["k"], "learned", ctx=state["ctx"])
        return {"idx": idx, "d2": d2, "flags": flags}
    if c["kind"] == "grad":
        loss, grads = kvb.mlp_backward(state["X"], state["near"], ctx=state["ctx"])
        return {"loss": loss, "grads": grads}
    if c["kind"] == "eigsh":
        e = kvb.eigsh(*state["csr"], nev=c["nev"], ncv=c["ncv"])
        return {"values": e.values, "residuals": e.residuals, "vectors": e.vectors}
    f, proj, coef = kvb.kolmogorov_solve(state["eigs"], state["P"], state["D"], state["g"])
    grads = [kvb.carre_du_champ(state["eigs"], state["P"], state["D"], f, x)[0] for x in state["X"]]
    return {"f": f, "proj": proj, "coef": coef, "grads": grads}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind in ("build", "learned"):
        n, m, k = case["n"], case["m"], case["k"]
        size = 4 * n * m + 8 * n * k + 4 * n                   # samples in; idx, d2, flags out
        flops = 3.0 * m * n * k                                # the distances that are returned
        if kind == "learned":
            h = (2 * m + 31) // 32 * 32
            return {"bytes": size, "flops": flops + 2.0 * n * (m * h + h * h + h * case["buckets"])}
        nnz = n * k
        size += 12 * n + 8 * (n + 1) + 8 * nnz + 16 * n        # b, rho, psi, rowptr, col, val, P, D out
        return {"bytes": size, "flops": flops + nnz * (2 * G * 3.0 + 30)}
    if kind == "grad":
        B, m, h1, h2, nb = case["batch"], case["m"], case["h1"], case["h2"], case["buckets"]
        w = m * h1 + h1 * h2 + h2 * nb
        return {"bytes": 4 * (B * m + B * case["ks"] + 2 * (w + h1 + h2 + nb)),
                "flops": 2.0 * B * (3 * w - m * h1)}
    if kind == "eigsh":
        n, nev, ncv = case["rows"] * case["cols"], case["nev"], case["ncv"]
        nnz = 69 * n
        # the matrix once a step, the basis once a step for the orthogonalisation, the vectors out
        return {"bytes": ncv * (8.0 * nnz + 24 * n) + 8.0 * n * ncv * ncv / 2 + 8.0 * n * nev,
                "flops": 2.0 * ncv * nnz + 4.0 * n * ncv * ncv / 2 + 2.0 * n * ncv * nev}
    n, nvec, coords = case["n"], case["nvec"], case["coords"]
    return {"bytes": 8.0 * n * (nvec + 5) + coords * 8.0 * n * (nvec + 5),
            "flops": 4.0 * n * nvec * 2 + coords * 2.0 * n * nvec * 8}


# ------------------------------------------------------------------ the same in float64
def _exact_knn(X, k):
    n = X.shape[0]
    Y = X - X.mean(0)
    sq = (Y * Y).sum(1)
    idx = torch.empty(n, k, dtype=torch.int64, device="cuda")
    d2 = torch.empty(n, k, dtype=torch.float64, device="cuda")
    keep = min(n, k + 8)
    step = max(1, (1 << 27) // n)
    for s in range(0, n, step):
        rows = torch.arange(s, min(n, s + step), device="cuda")
        score = torch.addmm(sq, Y[rows], Y.T, alpha=-2)
        score[rows - s, rows] = -math.inf
        near = score.topk(keep, dim=1, largest=False).indices.sort(dim=1).values
        d = torch.empty(rows.numel(), keep, dtype=torch.float64, device="cuda")
        part = max(1, (1 << 26) // (keep * X.shape[1]))
        for t in range(0, rows.numel(), part):
            d[t:t + part] = ((X[near[t:t + part]] - X[rows[t:t + part], None]) ** 2).sum(2)
        d[near == rows[:, None]] = -1
        d, at = d.sort(dim=1, stable=True)
        idx[rows], d2[rows] = near.gather(1, at)[:, :k], d[:, :k].clamp_min(0)
    return idx, d2


def _exact_build(c, seed):
    n, k, d = c["n"], c["k"], float(c["d"])
    alpha = -d / 4
    idx, d2 = _exact_knn(_samples(c["data"], n, c["m"], seed).double(), k)
    b = d2[:, 1:K0 + 1].sum(1).sqrt()
    row = torch.arange(n, device="cuda").repeat_interleave(k)
    col, dd = idx.reshape(-1), d2.reshape(-1)
    key = row * n + col
    if c["pattern"] == "union":
        key = torch.cat([key, col * n + row])
        dd = torch.cat([dd, dd])
    key, at = key.sort(stable=True)
    dd = dd[at]
    if c["pattern"] == "union":
        first = torch.ones_like(key, dtype=torch.bool)
        first[1:] = key[1:] != key[:-1]
        key, dd = key[first], dd[first]
    row, col = key // n, key % n

    def row_sum(v, r):
        return torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, r, v)

    def tune(rho, scale):
        x = dd / (rho[row] * rho[col])
        ln = np.log(E_MIN * scale) + np.arange(G) * (np.log(E_MAX * scale) - np.log(E_MIN * scale)) / (G - 1)
        e = np.exp(ln)
        chi = np.array([float(torch.exp(-x / v).sum()) for v in e])
        slope = np.diff(np.log(chi)) / np.diff(np.log(e))
        g = int(slope.argmax())
        return chi, float(e[g]), float(2 * slope[g])

    def kept(rho, e):
        K = torch.exp(-dd / (e * rho[row] * rho[col]))
        on = K > c["delta"] if c["delta"] > 0 else torch.ones_like(K, dtype=torch.bool)
        return row[on], col[on], K[on]

    chi_a, e_a, dim_a = tune(b, 1.0)
    r, j, K = kept(b, e_a)
    psi = row_sum(K, r) / (n * (math.pi * e_a * b * b) ** (d / 2))
    rho = 2 * psi ** BETA
    scale = 2.0 ** round(float((b.square().log().mean() - rho.square().log().mean()) / math.log(2)))
    chi_b, e_b, dim_b = tune(rho, scale)
    r, j, K = kept(rho, e_b)
    P = rho / 2
    q = row_sum(K, r) / P ** d
    Kt = K / (q[r] * q[j]) ** alpha
    D = row_sum(Kt, r)
    eye = (r == j).double()
    if c["out"] == "markov":
        val = Kt / D[r]
    elif c["out"] == "generator":
        val = (Kt / D[r] - eye) / (e_b * P[r] ** 2)
    else:
        S = P * D.sqrt()
        val = (Kt / (S[r] * S[j]) - eye / P[r] ** 2) / e_b
    if _varying(c):            # the caller's arrays keep their capacity
        val = torch.nn.functional.pad(val, (0, n * (2 * k - 1 if c["pattern"] == "union" else k) - val.numel()))
    return {"idx": None, "d2": d2, "flags": None, "b": b, "chi_a": chi_a, "e_a": e_a, "dim_a": dim_a, "rho": rho,
            "psi": psi, "scale_b": scale, "chi_b": chi_b, "e_b": e_b, "dim_b": dim_b, "rowptr": None, "col": None,
            "val": val, "P": P, "D": D}


def _exact_grad(c, state):
    W1, b1, W2, b2, W3, b3 = (t.double().requires_grad_() for t in _network(c, state["seed"]))
    z = torch.relu(torch.relu(state["X"].double() @ W1.T + b1) @ W2.T + b2) @ W3.T + b3
    target = torch.zeros_like(z).scatter_add_(1, state["near"].long(), torch.ones_like(state["near"],
                                                                                     dtype=torch.float64))
    loss = -(target / c["ks"] * torch.log_softmax(z, 1)).sum(1).mean()
    grads = torch.autograd.grad(loss, (W1, b1, W2, b2, W3, b3))
    return {"loss": float(loss), "grads": torch.cat([t.reshape(-1) for t in grads])}


def _exact_spectral(s):
    Y, lam = s["eigs"].vectors, torch.from_numpy(s["eigs"].values).cuda()
    S = s["P"] * s["D"].sqrt()
    n = S.numel()

    def coef(v):
        return Y @ (S * v)

    def at_samples(w):
        return (w @ Y) / S

    cg = coef(s["g"])[1:]
    f = (cg / lam[1:]) @ Y[1:] / S
    grads = []
    cf = coef(f)
    for x in s["X"]:
        cx = coef(x)
        U, V, LU, LV = at_samples(cf), at_samples(cx), at_samples(lam * cf), at_samples(lam * cx)
        grads.append(at_samples(0.5 * (lam * coef(U * V) - coef(LU * V) - coef(U * LV))))
    return {"f": f, "proj": cg @ Y[1:] / S, "coef": (cg / math.sqrt(n)).cpu().numpy(), "grads": grads}


def exact(case, seed):
    if case["kind"] == "build":
        return _exact_build(case, seed) if case["n"] <= EXACT_ROWS else None
    if case["kind"] == "grad":
        return _exact_grad(case, {**prepare(case, seed), "seed": seed})
    if case["kind"] == "spectral":
        return _exact_spectral(prepare(case, seed))
    return None       # the routed search returns no defined distances, the Krylov space no defined vectors
