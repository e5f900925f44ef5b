"""The calls of this package whose speed matters, as data: what a user's program
prepares, what one pass is, what it cannot do without, and what it should give.

``listed()`` names the fixed cases, ``draw(rng)`` gives more from the same
ranges, ``prepare(case, seed)`` makes the state a program holds before the call,
``run(state)`` is one pass through the public entry points, ``work(case)`` the
bytes and operations of a pass, and ``exact(case, seed)`` its floating results
in 64 bits with plain torch.

Kinds of case: ``pr`` (PageRank), ``bfs``, ``ppr`` (batched personalised
PageRank), ``train`` (a training step through the PPR solve: forward and edge
weight gradient), ``tc`` (triangle counts), ``bc`` (betweenness), ``multi``
(many small graphs in one launch).

A BFS parent is any in-neighbour one level up and may differ from run to run,
so passes that search return levels and per-root statistics; the parents are
computed all the same.
"""
import os

import torch

import graphgen as gg
import paper_2010_16012_amd as pp
from paper_2010_16012_amd import autotune

TUNED = os.path.join(os.path.dirname(os.path.abspath(autotune.__file__)), "tuned.json")
F = 0.85
DIRS = {"push": pp.PP_PUSH, "pull": pp.PP_PULL, "switch": pp.PP_SWITCH}


def listed():
    return [
        # a small graph ranked inside a larger program: launches and host time count
        {"name": "pr_pull_rmat10", "kind": "pr", "graph": "rmat", "scale": 10, "ef": 16, "weighted": False,
         "dir": "pull", "iters": 20},
        # the benchmark's own graph with its tuned settings
        {"name": "pr_pull_rmat22", "kind": "pr", "graph": "rmat", "scale": 22, "ef": 16, "weighted": False,
         "dir": "pull", "iters": 20},
        # the pushing form on a skewed graph of ordinary size
        {"name": "pr_push_rmat20", "kind": "pr", "graph": "rmat", "scale": 20, "ef": 16, "weighted": False,
         "dir": "push", "iters": 20},
        # uniform degrees, no hubs, an odd vertex count, untuned settings
        {"name": "pr_pull_er3m", "kind": "pr", "graph": "er", "n": 3000017, "ef": 8, "weighted": False,
         "dir": "pull", "iters": 20},
        # searches from a batch of roots with the direction chosen per level
        {"name": "bfs_switch_rmat20_x16", "kind": "bfs", "graph": "rmat", "scale": 20, "ef": 16, "roots": 16,
         "dir": "switch"},
        # pushing (top-down) searches, a few roots
        {"name": "bfs_push_rmat21_x4", "kind": "bfs", "graph": "rmat", "scale": 21, "ef": 16, "roots": 4,
         "dir": "push"},
        # a deep search: some two thousand levels, each a narrow frontier
        {"name": "bfs_grid", "kind": "bfs", "graph": "grid", "rows": 1000, "cols": 1031, "roots": 1, "dir": "switch"},
        # recommendations for a hundred sources at once; the second column tile is partial
        {"name": "ppr_pull_rmat18_k100", "kind": "ppr", "graph": "rmat", "scale": 18, "ef": 16, "dir": "pull",
         "k": 100, "k_tile": 64, "iters": 30},
        # one training step on edge weights: pushing forward, pulling adjoint, both to a tolerance
        {"name": "train_rmat16_k32", "kind": "train", "graph": "rmat", "scale": 16, "ef": 16, "k": 32, "k_tile": 32,
         "fwd": "push", "bwd": "pull"},
        # triangle counts of a skewed graph
        {"name": "tc_pull_rmat16", "kind": "tc", "graph": "rmat", "scale": 16, "ef": 16, "dir": "pull"},
        # betweenness sampled over 64 sources
        {"name": "bc_rmat16_s64", "kind": "bc", "graph": "rmat", "scale": 16, "ef": 16, "sources": 64,
         "fwd": "pull", "bwd": "pull"},
        # a batch of small graphs of very different sizes, ranked and searched in one launch
        {"name": "multi128", "kind": "multi", "graphs": 128, "lo": 8, "hi": 14, "dir": "pull"},
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _draw_graph(rng, lo, hi, kinds):
    """A graph of lo..hi vertices or so."""
    kind = rng.choice(kinds)
    n = _log_int(rng, lo, hi)
    if kind == "rmat":
        return {"graph": "rmat", "scale": max(1, (n - 1).bit_length() - 1), "ef": rng.randint(5, 16)}
    if kind == "er":
        return {"graph": "er", "n": n | 1, "ef": rng.randint(3, 8)}
    rows = max(2, int((n ** 0.5) * 2.0 ** rng.uniform(-1, 1)))
    return {"graph": "grid", "rows": rows, "cols": max(2, n // rows)}


def draw(rng):
    kind = rng.choice(["pr", "pr", "pr", "bfs", "bfs", "ppr", "train", "tc", "bc", "multi"])
    if kind == "pr":
        c = _draw_graph(rng, 500, 4000000, ["rmat", "rmat", "er", "grid"])
        size = (1 << c["scale"]) if c["graph"] == "rmat" else c.get("n", 0)
        return {"kind": "pr", **c, "weighted": 0 < size <= 1 << 17 and rng.random() < 0.5,
                "dir": rng.choice(["pull", "pull", "push"]), "iters": rng.randint(10, 30)}
    if kind == "bfs":
        c = _draw_graph(rng, 1000, 2000000, ["rmat", "rmat", "er"]) if rng.random() < 0.75 else \
            _draw_graph(rng, 1000, 500000, ["grid"])
        return {"kind": "bfs", **c, "roots": 1 if c["graph"] == "grid" else rng.randint(1, 16),
                "dir": rng.choice(["switch", "push", "pull"] if c["graph"] != "grid" else ["switch", "push"])}
    if kind == "ppr":
        d = rng.choice(["pull", "pull", "switch", "push"])
        return {"kind": "ppr", **_draw_graph(rng, 500, 60000 if d == "push" else 250000, ["rmat", "er", "grid"]),
                "dir": d, "k": _log_int(rng, 1, 100), "k_tile": rng.choice([8, 16, 32, 64]), "iters": 30}
    if kind == "train":
        return {"kind": "train", **_draw_graph(rng, 300, 60000, ["rmat", "er"]), "k": _log_int(rng, 2, 32),
                "k_tile": rng.choice([8, 16, 32]), "fwd": rng.choice(["pull", "push"]), "bwd": "pull"}
    if kind == "tc":
        return {"kind": "tc", **_draw_graph(rng, 500, 120000, ["rmat", "rmat", "er", "grid"]),
                "dir": rng.choice(["pull", "push"])}
    if kind == "bc":
        return {"kind": "bc", **_draw_graph(rng, 300, 70000, ["rmat", "er"]), "sources": _log_int(rng, 1, 64),
                "fwd": rng.choice(["pull", "push"]), "bwd": "pull"}
    return {"kind": "multi", "graphs": _log_int(rng, 4, 128), "lo": rng.randint(6, 9), "hi": rng.randint(10, 14),
            "dir": rng.choice(["pull", "push"])}


def _host(case, seed):
    if case["kind"] == "train":
        seed = 1  # training keeps its graph: the weights, sources and loss are new
    if case["graph"] == "rmat":
        return gg.rmat(case["scale"], case["ef"], seed=seed)
    if case["graph"] == "er":
        return gg.erdos_renyi(case["n"], case["ef"] * case["n"], seed=seed)
    return gg.grid(case["rows"], case["cols"], 0.05, seed=seed)


def _input(case, seed):
    """The host graph of a case and the vertices (roots or sources) it is asked about."""
    host = _host(case, seed)
    if case.get("weighted") or case["kind"] == "train":
        gg.with_weights(host, seed=seed + 1)
    want = case.get("roots") or case.get("k") or case.get("sources") or 0
    picks = gg.pick_vertices(host, want, seed=seed + 2) if want else None
    if case["graph"] == "grid" and case["kind"] == "bfs":
        # the deepest start is a corner: the first vertex with a neighbour
        picks[0] = int((host.out_degree() > 0).argmax())
    return host, picks


def _batch(case, seed):
    """The graphs of a batch: sizes by the case, edges by the seed."""
    scales = gg.uniform_int(case["graphs"], case["lo"], case["hi"], 1, stream=11)
    return [gg.rmat(int(sc), 16, seed=gg.rand_u64(seed, 12, i) >> 1) for i, sc in enumerate(scales)]


def prepare(case, seed):
    if case["kind"] == "multi":
        hosts = _batch(case, seed)
        autotune.apply(autotune.load_key(TUNED, autotune.multi_key(
            len(hosts), sum(h.n for h in hosts), sum(int(h.nnz) for h in hosts))))
        return {"case": case, "mg": pp.MultiGraph(hosts)}
    host, picks = _input(case, seed)
    tuned = autotune.load(TUNED, host.n, host.nnz)
    autotune.apply(tuned)
    # triangle counts read the rows as given; the other sweeps want the renumbered ones
    g = pp.Graph(host, relabel=case["kind"] != "tc")
    autotune.apply({})
    s = {"case": case, "g": g, "picks": picks, "dir": DIRS[case.get("dir", "pull")]}
    if case["kind"] == "bfs":
        s["run"] = pp.BfsRun(g)
        s["switch"] = (tuned.get("alpha", 14.0), tuned.get("beta", 24.0))
    elif case["kind"] == "train":
        s["w"] = torch.as_tensor(host.weights).cuda().requires_grad_(True)
        s["c"] = torch.as_tensor(gg.normal(host.n * case["k"], seed=seed + 3)).reshape(host.n, case["k"]).cuda()
    return s


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "pr":
        return pp.pagerank(s["g"], iters=case["iters"], f=F, direction=s["dir"])
    if kind == "bfs":
        stats = s["run"].run_many(s["picks"], s["dir"], *s["switch"])
        return {"level": s["run"].level, "levels": [st.levels for st in stats][:16],
                "reached": [st.reached for st in stats][:16], "edges": [st.edges_reached for st in stats][:16]}
    if kind == "ppr":
        return pp.ppr(s["g"], s["picks"], iters=case["iters"], f=F, k_tile=case["k_tile"], direction=s["dir"])[0]
    if kind == "train":
        X = pp.PPRFunction.apply(s["w"], s["g"], s["picks"], F, 300, 1e-6, case["k_tile"], DIRS[case["fwd"]],
                                 DIRS[case["bwd"]])
        return {"X": X, "grad": torch.autograd.grad(X, s["w"], s["c"])[0]}
    if kind == "tc":
        return pp.triangles(s["g"], s["dir"])
    if kind == "bc":
        return pp.betweenness(s["g"], s["picks"], DIRS[case["fwd"]], DIRS[case["bwd"]])
    x, level, _ = s["mg"].run(pr_iters=20, f=F, pr_dir=DIRS[case["dir"]], bfs_policy=pp.PP_SWITCH)
    return {"x": x, "level": level}


def _size(case):
    """Vertices and stored edges of a case, before duplicates are dropped."""
    if case["graph"] == "rmat":
        n = 1 << case["scale"]
        return n, 2 * case["ef"] * n
    if case["graph"] == "er":
        return case["n"], 2 * case["ef"] * case["n"]
    return case["rows"] * case["cols"], int(3.8 * case["rows"] * case["cols"])


def work(case):
    """Bytes: the adjacency and the state of every sweep (sweeps depend on one
    another, and a large adjacency does not stay on the chip between them)."""
    kind = case["kind"]
    if kind == "multi":
        scales = range(case["lo"], case["hi"] + 1)
        n = case["graphs"] * sum(1 << s for s in scales) / len(scales)
        nnz = 32 * n
        return {"bytes": 21 * (2 * nnz + 4 * n) + 12 * n, "flops": 20 * 2 * nnz}
    n, nnz = _size(case)
    if kind == "pr":
        per = (8 if case["weighted"] else 4) * nnz + 16 * n
        return {"bytes": case["iters"] * per, "flops": case["iters"] * 2 * nnz}
    if kind == "bfs":
        return {"bytes": case["roots"] * (4 * nnz + 12 * n), "flops": 0}
    if kind == "ppr":
        tiles = -(-case["k"] // case["k_tile"])
        return {"bytes": case["iters"] * (tiles * (4 * nnz + 4 * n) + 12 * n * case["k"]),
                "flops": case["iters"] * 2 * nnz * case["k"]}
    if kind == "train":
        # some 20 forward and 50 adjoint sweeps, then the gradient
        tiles = -(-case["k"] // case["k_tile"])
        return {"bytes": 70 * (tiles * 8 * nnz + 12 * n * case["k"]) + 12 * nnz, "flops": 70 * 2 * nnz * case["k"]}
    if kind == "tc":
        return {"bytes": 4 * nnz + 12 * n, "flops": 0}
    return {"bytes": 2 * 4 * nnz + 28.0 * n * case["sources"], "flops": 4.0 * nnz * case["sources"]}


# ------------------------------------------------------------- 64-bit results

def _edges(host):
    """Sources, targets (int64, on the device) and weights (FP64) of every stored edge."""
    deg = torch.as_tensor(host.out_degree()).cuda()
    src = torch.repeat_interleave(torch.arange(host.n, device="cuda"), deg)
    dst = torch.as_tensor(host.idx).cuda().long()
    w = None if host.weights is None else torch.as_tensor(host.weights).cuda().double()
    strength = deg.double() if w is None else torch.zeros(host.n, dtype=torch.float64, device="cuda").index_add_(0, src, w)
    inv = torch.where(strength > 0, 1.0 / strength, torch.zeros_like(strength))
    return src, dst, w, inv


def _f64():
    return float(torch.tensor(F, dtype=torch.float32))  # the entry points take f as float


def _exact_pr(hosts, iters):
    out = []
    for host in hosts:
        f = _f64()
        src, dst, w, inv = _edges(host)
        p = inv[src] if w is None else inv[src] * w
        x = torch.full((host.n,), 1.0 / host.n, dtype=torch.float64, device="cuda")
        for _ in range(iters):
            y = torch.full_like(x, (1.0 - f) / host.n)
            x = y.index_add_(0, dst, f * p * x[src])
        out.append(x)
    return torch.cat(out)


def _spread(src, dst, p, x):
    """y[dst] += p * x[src] over rows of columns, the edges in pieces that fit memory."""
    y = torch.zeros_like(x)
    piece = max(1, (1 << 27) // max(1, x.shape[1]))
    for a in range(0, len(src), piece):
        y.index_add_(0, dst[a:a + piece], p[a:a + piece, None] * x[src[a:a + piece]])
    return y


def _exact_ppr(host, picks, iters):
    f = _f64()
    src, dst, w, inv = _edges(host)
    p = f * (inv[src] if w is None else inv[src] * w)
    e = torch.zeros(host.n, len(picks), dtype=torch.float64, device="cuda")
    e[torch.as_tensor(picks).cuda().long(), torch.arange(len(picks), device="cuda")] = 1.0
    x = e
    for _ in range(iters):
        x = (1.0 - f) * e + _spread(src, dst, p, x)
    return x


def _exact_train(host, picks, c):
    f = _f64()
    x = _exact_ppr(host, picks, 130)
    src, dst, w, inv = _edges(host)
    p = inv[src] * w
    lam = c
    for _ in range(130):
        lam = c + f * _spread(dst, src, p, lam)
    ptl = _spread(dst, src, p, lam)
    grad = torch.empty(len(src), dtype=torch.float64, device="cuda")
    for a in range(0, len(src), 1 << 21):
        v, u = src[a:a + (1 << 21)], dst[a:a + (1 << 21)]
        grad[a:a + (1 << 21)] = f * inv[v] * (x[v] * (lam[u] - ptl[v])).sum(1)
    return {"X": x, "grad": grad}


def _exact_bc(host, picks):
    src, dst, _, _ = _edges(host)
    m = len(picks)
    at = (torch.as_tensor(picks).cuda().long(), torch.arange(m, device="cuda"))
    ones = torch.ones(len(src), dtype=torch.float64, device="cuda")
    dist = torch.full((host.n, m), -1, dtype=torch.int32, device="cuda")
    sigma = torch.zeros(host.n, m, dtype=torch.float64, device="cuda")
    dist[at], sigma[at] = 0, 1.0
    depth = 0
    while True:
        got = _spread(src, dst, ones, torch.where(dist == depth, sigma, 0.0))
        new = (dist < 0) & (got > 0)
        if not bool(new.any()):
            break
        depth += 1
        dist[new] = depth
        sigma = torch.where(new, got, sigma)
    delta = torch.zeros_like(sigma)
    for d in range(depth, 0, -1):
        share = torch.where(dist == d, (1.0 + delta) / sigma.clamp(min=1.0), 0.0)
        delta = torch.where(dist == d - 1, sigma * _spread(dst, src, ones, share), delta)
    delta[at] = 0.0
    return delta.sum(1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "multi":
        return {"x": _exact_pr(_batch(case, seed), 20), "level": None}
    if kind in ("bfs", "tc"):
        return None  # whole numbers
    host, picks = _input(case, seed)
    if kind == "pr":
        return _exact_pr([host], case["iters"])
    if kind == "ppr":
        return _exact_ppr(host, picks, case["iters"])
    if kind == "train":
        c = torch.as_tensor(gg.normal(host.n * case["k"], seed=seed + 3)).reshape(host.n, case["k"]).cuda().double()
        return _exact_train(host, picks, c)
    return _exact_bc(host, picks)
