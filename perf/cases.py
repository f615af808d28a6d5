"""What is timed: passes of the engine through its public entry points.

A case is a dict: ``kind`` names the entry point, (M, N, K) the problem, ``iters`` the DID
iterations of one pass, ``x`` the storage of X ("given": float32 column-major as the caller
holds it, "tiled": float32 in tile order, "bf16").

  solo    a handle the program keeps: ``did_iterate`` and ``did_factors``
  solve   one whole solve: ``did_init_ex``, ``did_iterate``, ``did_objective``,
          ``did_factors``, ``did_free``
  static  ``did_iterate_static`` on the caller's buffers
  batch   jobs of uneven shape advanced together: ``did_batch_*`` and ``did_factors``
  serve   jobs through the serving loop: ``did_server_*``

X holds products of U[0,1) factors with Gaussian noise, clipped at zero (the served jobs'
recipe); for the thin sets it is the product itself (the experiments' recipe).
"""

import math
import random

import numpy as np
import torch

import paper_1802_08938_amd as did

NOISE = 0.02


def listed():
    return [
        # the experiments' synthetic sets (M = 5, K = 3), the smallest: a run to convergence
        # takes a few hundred iterations of a problem of 2 MB, so latency is what counts
        dict(name="paper_1e5", kind="solo", x="given", M=5, N=100_000, K=3, iters=20),
        # the same sets at their largest: one stream over 3.2 GB per iteration
        dict(name="paper_1e8", kind="solo", x="given", M=5, N=100_000_000, K=3, iters=3),
        # a small dense problem (the planted test workload) iterated on a kept handle
        dict(name="planted_500x2000", kind="solo", x="given", M=500, N=2000, K=10, iters=20),
        # a set of images (MNIST's shape), as the image-like benchmark workload
        dict(name="image_784x70000", kind="solo", x="given", M=784, N=70_000, K=16, iters=10),
        # few samples with many features (UMist's shape): tall X
        dict(name="tall_10304x575", kind="solo", x="given", M=10_304, N=575, K=25, iters=5),
        # a whole solve of an odd shape, from the data to the factors and back to no state
        dict(name="solve_3809x2248", kind="solve", x="given", M=3809, N=2248, K=49, iters=20),
        # a mid-sized problem on a kept handle, X in tile order
        dict(name="tiled_1868x40000", kind="solo", x="tiled", M=1868, N=40_000, K=60, iters=5),
        # a slice of the large workload with X stored as bf16
        dict(name="bf16_5000x62500", kind="solo", x="bf16", M=5000, N=62_500, K=50, iters=5),
        # the large workload in the benchmark's configuration
        dict(name="large_5000x1e6", kind="solo", x="tiled", M=5000, N=1_000_000, K=50, iters=2),
        # the allocation-free call, one iteration at a time on the caller's buffers
        dict(name="static_600x9000", kind="static", x="given", M=600, N=9000, K=40, iters=1),
        # uneven jobs of the served distribution advanced together
        dict(name="batch_24", kind="batch", x="tiled", jobs=24, job_seed=5, iters=5),
        # jobs through the serving loop, from submission to release
        dict(name="serve_12", kind="serve", x="tiled", jobs=12, job_seed=7, iters=10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["thin", "solo", "solo", "solo", "solve", "static", "batch", "serve"])
    if kind == "thin":
        M, K = rng.choice([(5, 3), (5, 3), (rng.randint(2, 8), rng.randint(1, 4)), (rng.randint(9, 16), rng.randint(2, 4)),
                           (8, rng.randint(5, 8))])
        N = _log_int(rng, 100_000, 50_000_000)
        return dict(kind="solo", x="given", M=M, N=N, K=min(K, M), iters=3 if N > 5_000_000 else 20)
    if kind in ("batch", "serve"):
        return dict(kind=kind, x=rng.choice(["tiled", "tiled", "given", "bf16"]), jobs=rng.randint(4, 16),
                    job_seed=rng.randrange(1 << 30), iters=rng.randint(2, 10))
    x = rng.choice(["given", "tiled", "bf16"]) if kind == "solo" else "given"
    M = _log_int(rng, 100, 8000)
    N = _log_int(rng, 1000, 30_000 if kind == "static" else 200_000)
    K = rng.randint(5, 64)
    iters = 1 if kind == "static" else (10 if M * N < 10_000_000 else 5)
    return dict(kind=kind, x=x, M=M, N=N, K=K, iters=iters)


def _jobs(case):
    """Shapes of a case's jobs: the served workload's distribution."""
    rng = random.Random(case["job_seed"])
    out = []
    for _ in range(case["jobs"]):
        M, N = rng.randint(100, 4000), _log_int(rng, 1000, 200_000)
        out.append((M, N, min(rng.randint(5, 64), M, N), rng.randrange(1 << 31)))
    return out


def _data(M, N, K, seed):
    """X as a float32 (N, M) tensor, the column-major M x N."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    noise = 0.0 if M <= 16 else NOISE
    Bt = torch.rand((K, M), generator=g, device="cuda")
    X = torch.empty((N, M), device="cuda")
    step = max(1, (1 << 26) // M)
    for a in range(0, N, step):
        x = X[a:a + step]
        torch.matmul(torch.rand((len(x), K), generator=g, device="cuda"), Bt, out=x)
        if noise:
            x.add_(torch.randn(x.shape, generator=g, device="cuda"), alpha=noise).clamp_(min=0.0)
    return X


def _start(M, N, K, seed):
    """Initial factors U[0,1): B as (K, M) and C as (N, K), the column-major layouts."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + 1)
    return torch.rand((K, M), generator=g, device="cuda"), torch.rand((N, K), generator=g, device="cuda")


def _options(x):
    o = did.did_default_opts()
    o.x_dtype = did.DID_BF16 if x == "bf16" else did.DID_F32
    o.x_tiled = int(x == "tiled")
    o.borrow_x = int(x == "given")
    return o


class _State:
    """Handles and buffers of one case; gives the engine's objects back when it goes."""

    def __init__(self, case):
        self.case, self.handles, self.batch, self.server = case, [], None, None
        self.X, self.out, self.jobs = [], [], []

    def add(self, M, N, K, seed):
        X, (B, C) = _data(M, N, K, seed), _start(M, N, K, seed)
        torch.cuda.synchronize()  # the engine reads on its own stream
        self.handles.append(did.did_init_from_factors(X, M, N, K, B, C, _options(self.case["x"])))
        if self.case["x"] == "given":
            self.X.append(X)
        self.out.append((B, C))  # the factors are copied out here

    def __del__(self):
        if self.batch is not None:
            did.did_batch_free(self.batch)
        if self.server is not None:
            did.did_server_free(self.server)
        for h in self.handles:
            did.did_free(h)


def prepare(case, seed):
    s = _State(case)
    kind = case["kind"]
    if kind == "solo":
        s.add(case["M"], case["N"], case["K"], seed)
    elif kind == "batch":
        for M, N, K, js in _jobs(case):
            s.add(M, N, K, js + seed)
        s.batch = did.did_batch_create()
    elif kind == "serve":
        o = did.did_server_default_opts()
        o.max_iter, o.rel_tol, o.x_tiled = case["iters"], 0.0, int(case["x"] == "tiled")
        s.server = did.did_server_create(o)
        for M, N, K, js in _jobs(case):
            s.jobs.append((M, N, K, js + seed))
            s.X.append(_data(M, N, K, js + seed))
            s.out.append((torch.empty((K, M), device="cuda"), torch.empty((N, K), device="cuda")))
    else:
        M, N, K = case["M"], case["N"], case["K"]
        s.X.append(_data(M, N, K, seed))
        s.out.append(_start(M, N, K, seed))
        s.seed = seed
    torch.cuda.empty_cache()  # the engine allocates beside torch
    torch.cuda.synchronize()
    return s


def run(s):
    case, n = s.case, s.case["iters"]
    kind = case["kind"]
    if kind == "solo":
        B, C = s.out[0]
        did.did_iterate(s.handles[0], n)
        did.did_factors(s.handles[0], B, C)
        return B, C
    if kind == "static":
        B, C = s.out[0]
        did.did_iterate_static(s.X[0], case["M"], case["N"], case["K"], B, C, n)
        return B, C
    if kind == "solve":
        B, C = s.out[0]
        h = did.did_init_ex(s.X[0], case["M"], case["N"], case["K"], s.seed, _options(case["x"]))
        try:
            did.did_iterate(h, n)
            f = did.did_objective(h)
            did.did_factors(h, B, C)
        finally:
            did.did_free(h)
        return B, C, f
    if kind == "batch":
        for h in s.handles:
            did.did_batch_add(s.batch, h)
        did.did_batch_iterate(s.batch, n)
        for h, (B, C) in zip(s.handles, s.out):
            did.did_batch_remove(s.batch, h)
            did.did_factors(h, B, C)
        return s.out
    xt = did.DID_BF16 if case["x"] == "bf16" else did.DID_F32
    ids = [did.did_server_submit(s.server, X, M, N, K, js, xt) for X, (M, N, K, js) in zip(s.X, s.jobs)]
    left = 1
    while left:
        running, queued, _ = did.did_server_step(s.server)
        left = running + queued
    for j, (B, C) in zip(ids, s.out):
        did.did_server_result(s.server, j, B, C)
        did.did_server_release(s.server, j)
    return s.out


def work(case):
    """Each iteration reads X once and reads and writes the factors once; E, H, E' and W
    are 2 M N K operations each."""
    shapes = [j[:3] for j in _jobs(case)] if "jobs" in case else [(case["M"], case["N"], case["K"])]
    xb = 2 if case["x"] == "bf16" else 4
    n = case["iters"]
    return {"bytes": float(sum(n * (xb * M * N + 8 * K * (M + N)) for M, N, K in shapes)),
            "flops": float(sum(n * 8 * M * N * K for M, N, K in shapes))}


def _draws(count, seed, which):
    """The engine's documented initial draw: U[0,1) from splitmix64 keyed by (seed, which, i)."""
    with np.errstate(over="ignore"):
        def mix(z):
            z = z + np.uint64(0x9E3779B97F4A7C15)
            z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
            z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
            return z ^ (z >> np.uint64(31))

        key = mix(np.array([seed], np.uint64) ^ (np.array([which], np.uint64) * np.uint64(0xD1B54A32D192ED03)))
        z = mix(key + np.arange(1, count + 1, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15))
    return torch.from_numpy((z >> np.uint64(40)).astype(np.float64) * 2.0 ** -24).cuda()


def _iterate64(X, B, C, n):
    """n DID iterations in float64 from B (K, M) and C (N, K); returns B, C."""
    B, C = B.double(), C.double()
    K, (N, M) = B.shape[0], X.shape
    step = max(1, (1 << 27) // M)
    for _ in range(n):
        G, W, V = B @ B.t(), torch.zeros_like(B), torch.zeros((K, K), dtype=torch.float64, device=B.device)
        g = G.diagonal().tolist()
        for a in range(0, N, step):
            x, c = X[a:a + step].double(), C[a:a + step]
            h = ((x - c @ B) @ B.t().contiguous()).t().contiguous()
            ct = c.t().contiguous()
            for k in range(K):
                if g[k] > 0:
                    new = (ct[k] + h[k] / g[k]).clamp_(min=0.0)
                    h -= G[:, k:k + 1] * (new - ct[k])
                    ct[k] = new
            c.copy_(ct.t())
            e = x - c @ B
            W += ct @ e
            V += ct @ c
        d = torch.zeros_like(B)
        v = V.diagonal().tolist()
        for i in range(K):
            if v[i] > 0:
                new = (B[i] + (W[i] - V[i, :i] @ d[:i]) / v[i]).clamp_(min=0.0)
                d[i] = new - B[i]
        B = B + d
    return B, C


def _stored(X, x):
    return X.bfloat16().float() if x == "bf16" else X


def exact(case, seed):
    n = case["iters"]
    if "jobs" in case:
        out = []
        for M, N, K, js in _jobs(case):
            X = _stored(_data(M, N, K, js + seed), case["x"])
            if case["kind"] == "batch":
                B, C = _start(M, N, K, js + seed)
            else:
                B, C = _draws(K * M, js + seed, 1).view(K, M), _draws(N * K, js + seed, 2).view(N, K)
            out.append(_iterate64(X, B, C, n))
        return out
    M, N, K = case["M"], case["N"], case["K"]
    X = _stored(_data(M, N, K, seed), case["x"])
    if case["kind"] != "solve":
        return _iterate64(X, *_start(M, N, K, seed), n)
    B, C = _iterate64(X, _draws(K * M, seed, 1).view(K, M), _draws(N * K, seed, 2).view(N, K), n)
    return B, C, 0.5 * float((X.double() - C @ B).square().sum())
