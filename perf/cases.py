"""The calls a program makes of this library, at the sizes it makes them.

Every case goes through the package's public entry points:

* ``search``   -- ``henn_search_batch`` on an index the program holds, from a
                  single query to a full batch, on FP32, BF16 and FP8 rows;
                  ``captured`` replays the same search as a hipGraph with a
                  beam width and k of each request's own;
* ``build``    -- ``henn_build`` of a whole index, then ``export_layer`` of
                  every layer (what a program that builds and saves does);
* ``serve``    -- a continuous-batching ``Server`` run over a backlog;
* ``dynamic``  -- a sliding window: ``henn_insert`` of a batch, ``henn_delete``
                  of the oldest points, a search of the updated index.

Points and queries follow the distributions of ``workloads`` (Gaussian
mixtures, uniform, curve, power-law spectrum, skewed exponential), drawn on
the GPU from the case's seed alone.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2505_17368_amd as hn

BYTES = {"f32": 4, "bf16": 2, "fp8": 1}


def listed():
    return [
        # one lookup, nothing to batch it with: pure latency (the parity
        # workload's points and parameters)
        dict(name="one_query", op="search", data="uniform", n=10_000, d=32, metric="l2",
             graph="knn", degree=16, max_degree=32, root=0, storage="f32", nq=1, k=10, ef=32),
        # a handful of requests that came together, on the serving form's index
        dict(name="few_queries", op="search", data="gmm", clusters=100, sigma=0.3, n=300_000,
             d=128, metric="l2", graph="knn_sym", degree=32, max_degree=60, root=4096,
             storage="fp8", nq=48, k=10, ef=84),
        # the benchmark's own step: 10,000 queries on 1M x 128, tuned once
        dict(name="batch_fp8", op="search", data="gmm", clusters=100, sigma=0.3, n=1_000_000,
             d=128, metric="l2", graph="knn_sym", degree=32, max_degree=60, root=4096,
             storage="fp8", nq=10_000, k=10, ef=84, tuned=True),
        # plain FP32 rows with default settings; a width that fills no power
        # of two and a ragged batch
        dict(name="batch_f32_d100", op="search", data="gmm", clusters=100, sigma=0.3, n=200_003,
             d=100, metric="l2", graph="knn_sym", degree=32, max_degree=60, root=4096,
             storage="f32", nq=2_777, k=10, ef=64),
        # the throughput form: many requests, each with its own k and beam
        # width, replayed from a graph; an index past the one-byte visited tags
        dict(name="mixed_captured", op="search", data="gmm", clusters=1000, sigma=0.25,
             n=1_200_000, d=128, metric="l2", graph="knn_sym", degree=32, max_degree=60,
             root=4096, storage="fp8", nq=100_000, k=100, ef=128, captured=True),
        # embedding-like wide rows, inner product, a wide beam, greedy root
        dict(name="batch_ip_d768", op="search", data="spectral", n=60_000, d=768, metric="ip",
             graph="knn_sym", degree=32, max_degree=64, root=0, storage="bf16", nq=2_000, k=10,
             ef=256),
        # a small index: launches, allocations and synchronisations
        dict(name="build_small", op="build", data="uniform", n=10_000, d=32, metric="l2",
             graph="knn", degree=16, max_degree=32, root=0, storage="f32"),
        # the benchmark's index at half its points
        dict(name="build_sym", op="build", data="gmm", clusters=100, sigma=0.3, n=500_000,
             d=128, metric="l2", graph="knn_sym", degree=32, max_degree=60, root=4096,
             storage="fp8"),
        # embedding-like wide rows
        dict(name="build_ip_d768", op="build", data="spectral", n=60_000, d=768, metric="ip",
             graph="knn_sym", degree=32, max_degree=64, root=0, storage="bf16"),
        # the incremental-insertion graph of the skewed synthetic study
        dict(name="build_nsw", op="build", data="expskew", n=50_000, d=32, metric="l2",
             graph="nsw", degree=16, max_degree=32, root=0, storage="f32"),
        # a saturated request loop with mixed k and beam widths
        dict(name="serve", op="serve", data="gmm", clusters=100, sigma=0.3, n=300_000, d=128,
             metric="l2", graph="knn_sym", degree=32, max_degree=60, root=4096, storage="fp8",
             nq=40_000, k=50, ef=92, slots=8192, steps=128),
        # a window of recent points: a batch in, a batch out, then queries
        dict(name="dynamic", op="dynamic", data="gmm", clusters=100, sigma=0.3, n=60_000, d=128,
             metric="l2", graph="nsw", degree=16, max_degree=48, root=4096, storage="f32",
             nq=1_000, k=10, ef=128, count=3_000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["search"] * 5 + ["build"] * 3 + ["serve", "dynamic"])
    data = rng.choice(["gmm", "gmm", "gmm", "uniform", "expskew", "curve", "spectral"])
    d = _log_int(rng, 8, 768) if data == "spectral" else _log_int(rng, 16, 128)
    if rng.random() < 0.5 or data == "curve":
        d = max(8, d // 8 * 8)
    graph = rng.choice(["knn", "knn_sym", "knn_sym", "pruned_sym", "nsw"])
    if op == "dynamic":
        graph = "nsw"
    # the wide FP32 all-pairs pass and the insertion searches are the slow builds
    top = 40_000 if d > 128 else 60_000 if graph == "nsw" else 300_000
    n = _log_int(rng, 3_000, top)
    c = dict(op=op, data=data, n=n, d=d, metric="ip" if data == "spectral" else "l2", graph=graph,
             degree=rng.choice([16, 24, 32]), root=4096 if data == "gmm" else 0,
             storage=rng.choice(["f32", "bf16", "fp8"]))
    if data == "gmm":
        # a mixture needs a complete root that holds several points of every cluster
        root = n
        while root > 4096:
            root = root // 17
        c.update(clusters=max(2, min(1000, root // rng.randint(12, 36))),
                 sigma=rng.choice([0.25, 0.3]))
    c["max_degree"] = rng.choice([c["degree"] * 2 - 4, min(64, c["degree"] * 2)])
    if op in ("search", "dynamic", "serve"):
        c["k"] = rng.choice([1, 10, 10, 50, 100])
        c["ef"] = max(_log_int(rng, 16, 300), c["k"])
    if op == "search":
        c["nq"] = _log_int(rng, 1, 30_000 if d <= 128 else 4_000)
        c["captured"] = rng.random() < 0.2
    elif op == "serve":
        c.update(nq=_log_int(rng, 500, 20_000), slots=rng.choice([1024, 4096, 8192]),
                 steps=rng.choice([16, 64, 128]))
    elif op == "dynamic":
        c.update(nq=_log_int(rng, 1, 2_000), count=max(1, _log_int(rng, 50, 4_000) * n // 60_000))
    return c


# ----------------------------------------------------------------- inputs ---
def _gen(seed, word):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 16 + word)
    return g


def _basis(d, seed):
    g = torch.Generator()
    g.manual_seed(seed * 16 + 7)
    q, r = torch.linalg.qr(torch.randn(d, d, dtype=torch.float64, generator=g))
    return (q * torch.sign(torch.diagonal(r))[None, :]).cuda()


def _points(case, seed, word, count):
    """count rows of the case's distribution (its fixed part from the seed
    alone, the rows from (seed, word)), FP32 on the GPU."""
    data, d = case["data"], case["d"]
    g = _gen(seed, word)
    kw = dict(device="cuda", generator=g)
    if data == "uniform":
        return torch.rand(count, d, **kw)
    if data == "gmm":
        centres = torch.randn(case["clusters"], d, device="cuda", generator=_gen(seed, 0))
        lab = torch.randint(0, case["clusters"], (count,), **kw)
        return centres[lab].add_(torch.randn(count, d, **kw), alpha=case["sigma"])
    if data == "expskew":
        v = torch.rand(count, 1, **kw)
        x = torch.empty(count, d, device="cuda").exponential_(generator=g)
        return x / torch.pow(torch.tensor(32.0, device="cuda"), v)
    if data == "spectral":
        lam = torch.arange(1, d + 1, dtype=torch.float64, device="cuda") ** -0.8
        rot = (torch.sqrt(lam)[:, None] * _basis(d, seed).T).float()
        x = torch.randn(count, d, **kw) @ rot
        return x / x.norm(dim=1, keepdim=True)
    # curve: gaps 0.5^(i mod 40) along a unit-speed curve; queries (word > 1)
    # lie at the dense end of random periods
    half, period = d // 2, 40
    gf = _gen(seed, 0)
    omega = 2 * math.pi / (100.0 + 900.0 * torch.rand(half, dtype=torch.float64, device="cuda",
                                                      generator=gf))
    phase = 2 * math.pi * torch.rand(half, dtype=torch.float64, device="cuda", generator=gf)
    rho = 1.0 / (math.sqrt(half) * omega)
    gaps = 0.5 ** (torch.arange(case["n"], device="cuda", dtype=torch.float64) % period)
    t = torch.cumsum(gaps, 0) - gaps
    if word > 1:
        p = torch.randint(0, case["n"] // period, (count,), **kw)
        t = t[period * p + period - 1]
    ang = t[:, None] * omega[None, :] + phase[None, :]
    x = torch.empty(t.shape[0], d, dtype=torch.float64, device="cuda")
    x[:, 0::2] = rho * torch.cos(ang)
    x[:, 1::2] = rho * torch.sin(ang)
    x = x @ _basis(d, seed).T
    return (x + 1e-2 * torch.randn(x.shape, dtype=torch.float64, **kw)).float()


def _requests(case, seed):
    """Per-request k and beam width of the captured and serving forms."""
    rng = np.random.default_rng(seed + 6)
    k, ef, nq = case["k"], case["ef"], case["nq"]
    if case["op"] == "serve":
        ks, efs = [min(10, k), k], [max(1, ef - 8), max(1, ef - 4), ef]
    else:
        ks, efs = [1, min(10, k), k], [max(1, ef // 4), max(1, ef // 2), ef]
    return (rng.choice(np.array(ks, dtype=np.int32), nq),
            rng.choice(np.array(efs, dtype=np.int32), nq))


def _build_args(case):
    return dict(metric=case["metric"], graph=case["graph"], degree=case["degree"],
                max_degree=case["max_degree"], storage=case["storage"],
                root_complete_max=case["root"])


def prepare(case, seed):
    X = _points(case, seed, 1, case["n"])
    s = dict(case=case, X=X)
    op = case["op"]
    if op == "build":
        return s
    idx = hn.henn_build(X, **_build_args(case))
    s["idx"] = idx
    if op == "search":
        Q = s["Q"] = _points(case, seed, 2, case["nq"])
        if case.get("captured"):
            k, ef = _requests(case, seed)
            k, ef = torch.from_numpy(k).cuda(), torch.from_numpy(ef).cuda()
            s["graph"] = hn.SearchGraph(idx, Q, k=case["k"], ef=case["ef"], k_arr=k, ef_arr=ef,
                                        k_max=case["k"], ef_max=case["ef"])
        elif case.get("tuned"):
            hn.henn_autotune(idx, Q, k=case["k"], ef=case["ef"])
        del s["X"]
    elif op == "serve":
        s["Q"] = _points(case, seed, 2, case["nq"]).cpu().numpy()
        s["k"], s["ef"] = _requests(case, seed)
        s["tags"] = np.arange(case["nq"], dtype=np.int64)
        s["srv"] = hn.Server(idx, max_slots=case["slots"], pool_bytes=128 << 20,
                             k_max=case["k"], ef_max=case["ef"], steps_per_tick=case["steps"])
        del s["X"]
    else:
        s["Q"] = _points(case, seed, 2, case["nq"])
        # as many new points as the window holds, and some: a vector comes
        # back only when its earlier copy has left
        batches = -(-case["n"] // case["count"]) + 2
        s["new"] = (X[torch.randperm(case["n"], device="cuda", generator=_gen(seed, 4))]
                    if case["data"] == "curve" else
                    _points(case, seed, 3, min(batches * case["count"], 2 * case["n"])))
        s["at"], s["oldest"] = 0, 0
        del s["X"]
    return s


def run(s):
    case = s["case"]
    op = case["op"]
    if op == "search":
        if "graph" in s:
            ids, dist = s["graph"].launch()
        else:
            ids, dist = hn.henn_search_batch(s["idx"], s["Q"], k=case["k"], ef=case["ef"])
        return {"ids": ids, "dist": dist}
    if op == "build":
        idx = hn.henn_build(s["X"], **_build_args(case))
        layers = [idx.export_layer(i) for i in range(idx.num_layers)]
        idx.free()
        return {"ids": [a for a, _ in layers], "adj": [b for _, b in layers]}
    if op == "serve":
        srv, nq, k = s["srv"], case["nq"], case["k"]
        ids = np.empty((nq, k), dtype=np.int32)
        dist = np.empty((nq, k), dtype=np.float32)
        srv.submit_batch(s["Q"], s["k"], s["ef"], s["tags"])
        done = 0
        while done < nq:
            srv.tick()
            t, i, x = srv.poll()
            if len(t):
                ids[t], dist[t] = i, x
                done += len(t)
        return {"ids": ids, "dist": dist}
    c, new = case["count"], s["new"]
    if s["at"] + c > new.shape[0]:
        s["at"] = 0
    hn.henn_insert(s["idx"], new[s["at"]:s["at"] + c])
    hn.henn_delete(s["idx"], np.arange(s["oldest"], s["oldest"] + c, dtype=np.int32))
    s["at"] += c
    s["oldest"] += c
    ids, dist = hn.henn_search_batch(s["idx"], s["Q"], k=case["k"], ef=case["ef"])
    return {"ids": ids, "dist": dist}


# ------------------------------------------------------------------- work ---
def work(case):
    """Model counts, not the code's own.  Search: a beam of ef expands about
    ef nodes and evaluates about degree new rows at each; an expansion reads
    one adjacency row, an evaluation one stored row (read together by all
    queries, no row need be read more than once), the precision forms re-read
    4k rows in FP32.  All-pairs graphs: each unordered pair's distance once.
    Insertion graphs: one search of beam 256 a point."""
    n, d, R = case["n"], case["d"], case["degree"]
    M = R if case["graph"] == "knn" else case["max_degree"]
    row = d * BYTES[case["storage"]]
    op = case["op"]

    def search(nq, ef, k, b):
        rows = ef * R
        rr = 0 if b == 4 * d else 4 * k * 4 * d
        return (min(nq * (ef * M * 4 + rows * b), n * (M * 4 + b)) + nq * (rr + 4 * d + 8 * k),
                nq * rows * 2 * d)

    def graph(points):
        if case["graph"] == "nsw":
            b, f = search(points, 256, R, 4 * d)
            return b, f
        return 4 * n * d + 4 * n * M, float(n) * n * d

    if op == "build":
        b, f = graph(n)
        return {"bytes": b + n * row + 4 * n * M, "flops": f}
    b, f = search(case["nq"], case["ef"], case["k"], row)
    if op == "dynamic":
        gb, gf = graph(case["count"])
        b, f = b + gb, f + gf
    return {"bytes": b, "flops": f}


# ------------------------------------------------------------------ exact ---
def exact(case, seed):
    """Distances of the true k nearest, in 64 bits.  A search returns those its
    beam reaches, so this is only given where it reaches nearly all of them:
    symmetric graphs and a beam of some width on mixtures with a complete root
    or on the spectral data.  Ids have no such value."""
    n, d = case["n"], case["d"]
    if case["op"] not in ("search", "serve") or case["data"] not in ("gmm", "spectral"):
        return None
    if case["graph"] not in ("knn_sym", "pruned_sym") or case["ef"] < 48:
        return None
    nq = case["nq"]
    if float(nq) * n * d > 3e12:
        return None
    X = _points(case, seed, 1, n).double()
    Q = _points(case, seed, 2, nq).double()
    kmax = case["k"]
    kk = min(kmax, n)
    x2 = (X * X).sum(1)
    out = torch.full((nq, kmax), math.inf, dtype=torch.float64, device="cuda")
    step = max(1, int(2e8) // n)
    for b in range(0, nq, step):
        q = Q[b:b + step]
        g = q @ X.T
        if case["metric"] == "ip":
            out[b:b + step, :kk] = torch.topk(-g, kk, largest=False).values
        else:
            near = torch.topk(x2[None, :] - 2 * g, kk, largest=False).indices
            for j in range(kk):  # the difference form: nothing cancels
                out[b:b + step, j] = (q - X[near[:, j]]).square().sum(1)
    if case.get("captured") or case["op"] == "serve":
        k = torch.from_numpy(_requests(case, seed)[0]).cuda()
        out[torch.arange(kmax, device="cuda")[None, :] >= k[:, None]] = math.inf
    out = out.sort(1).values
    return {"ids": None, "dist": out.cpu().numpy() if case["op"] == "serve" else out}
