"""The calls whose speed matters to a user of this framework, as measurable cases.

A case is a dict of plain values; prepare() makes what a program has in hand
before the call (graphs, plans, weights), run() is one call through the public
entry points, work() the bytes and operations such a call cannot do without,
exact() the same results in 64 bits from plain torch.

The graph families are those of gen/ (uniform random digraphs, 4-neighbour
grids, R-MAT), drawn here on the GPU so that the large ones are quick to make.
"""
import math
import random

import torch

import paper_1812_10499_amd as sp

# ---------------------------------------------------------------- the cases


def listed():
    return [
        # one query on a small graph: a call made in a loop, where latency is everything
        dict(name="solve_random_1k", kind="solve", family="random", n=1003, degree=8,
             weights="int", wmax=100),
        # the framework's small benchmark graph
        dict(name="solve_random_4k", kind="solve", family="random", n=4096, degree=8,
             weights="int", wmax=100),
        # one query on an ordinary graph with real weights, an odd vertex count
        dict(name="solve_random_150k_f32", kind="solve", family="random", n=150001, degree=8,
             weights="unit"),
        # a road-like network: long diameter, thousands of small rounds
        dict(name="solve_grid_1024", kind="solve", family="grid", rows=1024, cols=1024,
             weights="int", wmax=1000),
        # the headline: a large skewed graph
        dict(name="solve_rmat_22", kind="solve", family="rmat", scale=22, edge_factor=16,
             weights="int", wmax=255),
        # one source, one destination: the rounds stop when the target is fixed
        dict(name="target_rmat_18", kind="target", family="rmat", scale=18, edge_factor=16,
             weights="int", wmax=255),
        # many graphs of mixed sizes, one query each, in one call
        dict(name="batch_256_f32", kind="batch", count=256, nmin=1000, nmax=200000, degree=8),
        # a query server: a recorded plan of 64 sources on one small graph, replayed
        dict(name="plan_64_random_4k", kind="plan", family="random", n=4001, degree=8,
             weights="int", wmax=100, sources=64),
        # a training step on a grid (new weights, 64 sources forward, backward)
        dict(name="train_grid_512", kind="train", family="grid", rows=512, cols=512,
             weights="half", sources=64),
        # a training step on an unstructured graph with few sources
        dict(name="train_random_30k", kind="train", family="random", n=30011, degree=8,
             weights="unit", sources=16),
        # building a large skewed graph from edges in device memory
        dict(name="build_rmat_20", kind="build", family="rmat", scale=20, edge_factor=16,
             weights="int", wmax=255),
        # building an ordinary graph with real weights, odd sizes
        dict(name="build_random_100k_f32", kind="build", family="random", n=100003, degree=8,
             weights="unit"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges."""
    kind = rng.choice(["solve", "solve", "solve", "target", "batch", "plan", "train", "train",
                       "build", "build"])
    case = dict(kind=kind)
    if kind == "batch":
        nmin = _log_int(rng, 100, 4000)
        case.update(count=_log_int(rng, 8, 128), nmin=nmin,
                    nmax=_log_int(rng, 2 * nmin, 200000), degree=rng.randint(3, 10))
        return case
    if kind == "train":
        case["sources"] = _log_int(rng, 3, 64)
        if rng.random() < 0.5:
            case.update(family="grid", rows=_log_int(rng, 30, 512), cols=_log_int(rng, 30, 512),
                        weights="half")
        else:
            case.update(family="random", n=_log_int(rng, 500, 50000), degree=rng.randint(3, 10),
                        weights="unit")
        return case
    if kind == "plan":
        case["sources"] = _log_int(rng, 5, 128)
        if rng.random() < 0.3:
            case.update(family="grid", rows=_log_int(rng, 10, 90), cols=_log_int(rng, 10, 90))
        else:
            case.update(family="random", n=_log_int(rng, 200, 20000), degree=rng.randint(3, 12))
    else:
        family = rng.choice(["random", "random", "grid", "rmat"])
        if kind == "target" and family == "grid":
            family = "rmat"
        case["family"] = family
        if family == "random":
            case.update(n=_log_int(rng, 300, 500000), degree=rng.randint(3, 12))
        elif family == "grid":
            case.update(rows=_log_int(rng, 16, 700), cols=_log_int(rng, 16, 700))
        else:
            case.update(scale=rng.randint(10, 20), edge_factor=rng.randint(6, 16))
    case["weights"] = rng.choice(["int", "int", "unit"]) if kind != "target" else "int"
    if case["weights"] == "int":
        case["wmax"] = 1000 if case["family"] == "grid" else rng.choice([100, 255])
    return case


# --------------------------------------------------------------- the inputs


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _ints(g, lo, hi, size):
    return torch.randint(lo, hi, (size,), generator=g, device="cuda", dtype=torch.int32)


def _random_edges(g, n, m):
    src = _ints(g, 0, n, m)
    dst = (src + _ints(g, 1, n, m)) % n if n > 1 else src.clone()
    return src, dst.to(torch.int32)


def _grid_edges(rows, cols):
    v = torch.arange(rows * cols, device="cuda", dtype=torch.int32)
    r, c = v // cols, v % cols
    src = torch.stack([v] * 4, 1)
    dst = torch.stack([v - cols, v + cols, v - 1, v + 1], 1)
    ok = torch.stack([r > 0, r < rows - 1, c > 0, c < cols - 1], 1)
    return src[ok], dst[ok]


def _rmat_edges(g, scale, m):
    src = torch.zeros(m, device="cuda", dtype=torch.int32)
    dst = torch.zeros(m, device="cuda", dtype=torch.int32)
    for _ in range(scale):  # quadrants of probability .57, .19, .19, .05
        u = torch.rand(m, generator=g, device="cuda")
        low = u >= 0.76
        src = 2 * src + low
        dst = 2 * dst + (((u >= 0.57) & ~low) | (u >= 0.95))
    relabel = torch.randperm(1 << scale, generator=g, device="cuda").to(torch.int32)
    return relabel[src], relabel[dst]


def _weights(g, case, m):
    kind = case["weights"]
    if kind == "int":
        return _ints(g, 1, case["wmax"] + 1, m)
    if kind == "unit":  # (0, 1], multiples of 2^-24
        return (_ints(g, 0, 1 << 24, m) + 1).to(torch.float32) * 2.0 ** -24
    return 0.5 + _ints(g, 0, (1 << 23) + 1, m).to(torch.float32) * 2.0 ** -23  # [0.5, 1.5]


def _size(case):
    """(vertices, edges) of a single-graph case."""
    if case["family"] == "random":
        return case["n"], case["n"] * case["degree"]
    if case["family"] == "grid":
        r, c = case["rows"], case["cols"]
        return r * c, 2 * (r * (c - 1) + c * (r - 1))
    return 1 << case["scale"], case["edge_factor"] << case["scale"]


def _edges(g, case):
    n, m = _size(case)
    if case["family"] == "random":
        src, dst = _random_edges(g, n, m)
    elif case["family"] == "grid":
        src, dst = _grid_edges(case["rows"], case["cols"])
    else:
        src, dst = _rmat_edges(g, case["scale"], m)
    return n, src, dst, _weights(g, case, m)


def _source(case, n, src):
    """A grid's centre, an R-MAT graph's vertex of largest out-degree, else vertex 0."""
    if case["family"] == "grid":
        return (case["rows"] // 2) * case["cols"] + case["cols"] // 2
    if case["family"] == "rmat":
        deg = torch.bincount(src, minlength=n)
        return int((deg == deg.max()).nonzero()[0])
    return 0


def _distinct(g, n, count):
    return torch.randperm(n, generator=g, device="cuda")[:count].tolist()


def _batch_inputs(case, seed):
    """One (n, src, dst, w, source) per instance."""
    g = _generator(seed)
    sizes = random.Random(case["count"])  # the sizes are the case's own, the rest the seed's
    out = []
    for _ in range(case["count"]):
        n = sizes.randint(case["nmin"], case["nmax"])
        src, dst = _random_edges(g, n, n * case["degree"])
        w = _weights(g, dict(weights="unit"), n * case["degree"])
        out.append((n, src, dst, w, n // 3))
    return out


def _train_inputs(case, seed):
    g = _generator(seed)
    n, src, dst, w = _edges(g, case)
    sources = _distinct(g, n, case["sources"])
    grad = torch.randn(len(sources), n, generator=g, device="cuda")
    return n, src, dst, w, sources, grad


# ------------------------------------------------------------- the programs


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        inputs = _batch_inputs(case, seed)
        return dict(kind=kind, graphs=[sp.Graph(*x[:4]) for x in inputs],
                    which=list(range(len(inputs))), sources=[x[4] for x in inputs])
    if kind == "train":
        n, src, dst, w, sources, grad = _train_inputs(case, seed)
        return dict(kind=kind, graph=sp.Graph(n, src, dst, w), w=w.requires_grad_(),
                    sources=sources, grad=grad)
    g = _generator(seed)
    n, src, dst, w = _edges(g, case)
    if kind == "build":
        return dict(kind=kind, n=n, src=src, dst=dst, w=w)
    graph = sp.Graph(n, src, dst, w)
    if kind == "plan":
        sources = _distinct(g, n, case["sources"])
        return dict(kind=kind, plan=sp.Plan([graph], [0] * len(sources), sources))
    state = dict(kind=kind, graph=graph, source=_source(case, n, src))
    if kind == "target":  # a vertex with edges, so usually a reachable one
        state["target"] = int(dst[dst.numel() // 2])
    return state


def run(state):
    kind = state["kind"]
    if kind == "solve":
        cost, pred, _ = sp.solve(state["graph"], state["source"])
        return cost, pred
    if kind == "target":
        return sp.solve_target(state["graph"], state["source"], state["target"])[0]
    if kind == "batch":
        cost, pred, _ = sp.solve_batch(state["graphs"], state["which"], state["sources"])
        return cost, pred
    if kind == "plan":
        return state["plan"].run()
    if kind == "train":
        cost = sp.shortest_paths(state["w"], state["graph"], state["sources"], order="coo")
        (gw,) = torch.autograd.grad(cost, state["w"], state["grad"])
        return cost.detach(), gw
    graph = sp.Graph(state["n"], state["src"], state["dst"], state["w"])
    return dict(graph.arrays(), perm=graph.perm)


def work(case):
    """A solve reads each edge's head and weight and each vertex's offset once and
    writes cost and parent per query; one add per edge and query."""
    if case["kind"] == "batch":
        n = case["count"] * (case["nmin"] + case["nmax"]) // 2
        m = n * case["degree"]
        return dict(bytes=8 * m + 12 * n, flops=m)
    n, m = _size(case)
    if case["kind"] == "build":  # three words per edge in, seven out; three per vertex out
        return dict(bytes=40 * m + 12 * n, flops=0)
    if case["kind"] == "target":  # no parents
        return dict(bytes=8 * m + 8 * n, flops=m)
    s = case.get("sources", 1)
    if case["kind"] == "train":  # weights in, gradient out, loss coefficients in, costs out
        return dict(bytes=12 * m + 4 * n + 8 * n * s, flops=s * (m + n))
    return dict(bytes=8 * m + 4 * n + 8 * n * s, flops=s * m)


# ------------------------------------------------------- the same in 64 bits


def _bellman_ford(n, src, dst, w, sources, dtype, inf):
    """Costs [S, n] by relaxing every edge until nothing changes."""
    src, dst, w = src.long(), dst.long(), w.to(dtype)
    cost = torch.full((len(sources), n), inf, dtype=dtype, device="cuda")
    cost[torch.arange(len(sources), device="cuda"), torch.tensor(sources, device="cuda")] = 0
    index = dst.expand(len(sources), -1)
    step = 0
    while True:
        cand = cost[:, src] + w
        new = cost.scatter_reduce(1, index, cand, "amin")
        step += 1
        if step % 16 == 0 and torch.equal(new, cost):
            return new
        cost = new


def _costs(n, src, dst, w, sources):
    if w.dtype == torch.int32:
        far = 1 << 40
        cost = _bellman_ford(n, src, dst, w, sources, torch.int64, far)
        return torch.where(cost >= far, torch.full_like(cost, 2 ** 31 - 1), cost)
    return _bellman_ford(n, src, dst, w, sources, torch.float64, float("inf"))


def _gradient(n, src, dst, w, sources, grad):
    """Sums of grad over the subtrees of the shortest-path trees, per edge in
    input order.  The trees are those of float32 costs (a tie is broken by the
    edge's place in the order by tail); None if a vertex has no tight in-edge
    from a cheaper vertex."""
    s = len(sources)
    cost = _bellman_ford(n, src, dst, w, sources, torch.float32, float("inf"))
    order = torch.sort(src, stable=True)[1]
    a, b, wk = src[order].long(), dst[order].long(), w[order]
    total = torch.zeros(src.numel(), dtype=torch.float64, device="cuda")
    for i in range(s):
        c = cost[i]
        tight = (c[a] + wk == c[b]) & (c[a] < c[b])
        ids = torch.arange(a.numel(), device="cuda")[tight]
        par = torch.full((n,), a.numel(), dtype=torch.int64, device="cuda")
        par = par.scatter_reduce(0, b[tight], ids, "amin")
        reach = c < float("inf")
        has = par < a.numel()
        reach[sources[i]] = False
        if bool((reach & ~has).any()):
            return None
        v = reach.nonzero()[:, 0]
        up = torch.arange(n, device="cuda")
        up[v] = a[par[v]]
        depth = torch.zeros(n, dtype=torch.int64, device="cuda")
        depth[v] = 1
        jump = up.clone()
        while True:  # pointer doubling
            d2 = depth + depth[jump]
            if torch.equal(d2, depth):
                break
            depth, jump = d2, jump[jump]
        acc = torch.where(c < float("inf"), grad[i].double(), torch.zeros((), dtype=torch.float64,
                                                                         device="cuda"))
        by = torch.sort(depth[v], descending=True, stable=True)
        counts = torch.bincount(depth[v]).flip(0).tolist() if v.numel() else []
        at = 0
        for k in counts:
            level = v[by[1][at:at + k]]
            acc.index_add_(0, up[level], acc[level])
            at += k
        total.index_add_(0, par[v], acc[v])
    out = torch.empty_like(total)
    out[order] = total
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("build", "target"):
        return None
    if kind == "batch":
        inputs = _batch_inputs(case, seed)
        base, src, dst, sources = 0, [], [], []
        for n, a, b, _, s in inputs:
            src.append(a + base)
            dst.append(b + base)
            sources.append(base + s)
            base += n
        w = torch.cat([x[3] for x in inputs])
        src, dst = torch.cat(src), torch.cat(dst)
        # one search over the disjoint union from all the sources at once
        root = torch.full((len(sources),), base, dtype=torch.int32, device="cuda")
        src = torch.cat([src, root])
        dst = torch.cat([dst, torch.tensor(sources, dtype=torch.int32, device="cuda")])
        w = torch.cat([w, torch.zeros(len(sources), device="cuda")])
        return _costs(base + 1, src, dst, w, [base])[0, :base], None
    if kind == "train":
        n, src, dst, w, sources, grad = _train_inputs(case, seed)
        return _costs(n, src, dst, w, sources), _gradient(n, src, dst, w, sources, grad)
    g = _generator(seed)
    n, src, dst, w = _edges(g, case)
    if kind == "plan":
        return _costs(n, src, dst, w, _distinct(g, n, case["sources"])).reshape(-1), None
    return _costs(n, src, dst, w, [_source(case, n, src)])[0], None
