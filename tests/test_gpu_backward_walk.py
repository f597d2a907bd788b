"""The tree pass of the backward on the shapes where it branches: chains,
vertices with one, two, three and many children, out-lists around the length
one lane scans alone, in-lists past the ones held in registers, several
instances and graphs, and pred arrays no solver wrote (stray trees, parent
cycles, entries that name another vertex's edge or none)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sp():
    import paper_1812_10499_amd as sp
    assert torch.cuda.is_available()
    return sp


def tree_grad(n, off, dst, root, pred, gcost, grad):
    """Adds one instance's gradient to grad, in float32 and the fixed order:
    a vertex's children in edge order."""
    order, at = [root], 0
    kids = {}
    while at < len(order):
        x = order[at]
        at += 1
        ks = [e for e in range(off[x], off[x + 1]) if dst[e] != root and pred[dst[e]] == e]
        kids[x] = ks
        order += [int(dst[e]) for e in ks]
    acc = {}
    for x in reversed(order):
        s = np.float32(gcost[x])
        for e in kids[x]:
            s = np.float32(s + acc[int(dst[e])])
        acc[x] = s
    for x in order:
        for e in kids[x]:
            grad[e] = np.float32(grad[e] + acc[int(dst[e])])


def random_tree(rng, n, kind):
    """Edges of a tree over a random numbering, and some more."""
    ids = rng.permutation(n)
    if kind == "chain":
        up = np.arange(n - 1)
    elif kind == "binary":
        up = np.arange(n - 1) // 2
    elif kind == "ternary":
        up = np.arange(n - 1) // 3
    elif kind == "star":
        up = np.where(np.arange(n - 1) % 5 == 0, 0, np.arange(n - 1) // 7)
    elif kind in ("scan15", "scan16", "scan17"):
        up = np.arange(n - 1) // int(kind[4:])
    else:
        up = (rng.random(n - 1) * np.arange(1, n)).astype(np.int64)
    src, dst = ids[up], ids[1:]
    if kind not in ("scan15", "scan16", "scan17"):
        extra = rng.integers(0, n, (2, 3 * n))
        if kind == "star":
            extra[1, : n] = ids[n // 2]  # a vertex of many in-edges
        src, dst = np.concatenate([src, extra[0]]), np.concatenate([dst, extra[1]])
    return src.astype(np.int32), dst.astype(np.int32), int(ids[0])


def tree_pred(rng, n, off, dst, root, spoil):
    """Parent entries of a random spanning tree of what root reaches; spoil
    rewrites some of them."""
    pred = np.full(n, -1, np.int32)
    seen, order, at = {root}, [root], 0
    while at < len(order):
        x = order[at]
        at += 1
        for e in rng.permutation(np.arange(off[x], off[x + 1])):
            y = int(dst[e])
            if y not in seen:
                seen.add(y)
                pred[y] = e
                order.append(y)
    m = len(dst)
    if spoil:
        some = rng.integers(0, n, max(2, n // 20))
        pred[some] = rng.integers(-3, m + 3, len(some))      # mostly another vertex's edge
        for e in rng.integers(0, m, max(2, n // 10)):
            pred[dst[e]] = e                                  # any in-edge: cycles, stray trees
        pred[root] = rng.integers(0, m)
    return pred


@pytest.mark.parametrize("spoil", [False, True])
@pytest.mark.parametrize("kind,n,count", [
    ("random", 2, 1), ("chain", 3, 2), ("chain", 1500, 1), ("binary", 1023, 9),
    ("ternary", 1093, 3), ("star", 2000, 17), ("scan15", 1000, 2), ("scan16", 1000, 2),
    ("scan17", 1000, 2), ("random", 257, 70), ("random", 3001, 5)])
def test_walk_matches_ordered_sums(sp, kind, n, count, spoil):
    rng = np.random.default_rng(n + count)
    src, dst, root = random_tree(rng, n, kind)
    w = rng.integers(1, 9, len(src)).astype(np.float32)
    A = sp.Graph(n, src, dst, w)
    B = sp.Graph(4, np.array([0, 1], np.int32), np.array([1, 3], np.int32),
                 np.array([1, 2], np.float32))
    graphs, inst, sources, preds, gcosts = [B, A], [], [], [], []
    want = [np.zeros(B.m, np.float32), np.zeros(A.m, np.float32)]
    for i in range(count):
        g = 0 if i == 1 else 1
        G = graphs[g]
        arr = G.arrays()
        off, hd = arr["out_off"].cpu().numpy(), arr["out_dst"].cpu().numpy()
        r = 0 if g == 0 else root if i % 3 else int(rng.integers(0, n))
        pred = tree_pred(rng, G.n, off, hd, r, spoil and g == 1)
        gc = rng.standard_normal(G.n).astype(np.float32)
        inst.append(g)
        sources.append(r)
        preds.append(pred)
        gcosts.append(gc)
        tree_grad(G.n, off, hd, r, pred, gc, want[g])
    p = torch.from_numpy(np.concatenate(preds)).cuda()
    gc = torch.from_numpy(np.concatenate(gcosts)).cuda()
    for _ in range(2):
        got = sp.backward(graphs, inst, sources, p, gc).cpu().numpy()
        assert np.array_equal(got, np.concatenate(want))


@pytest.mark.parametrize("count", [63, 80])
def test_walk_shared_by_an_xcds_waves(sp, count):
    """Around the line where each tree stays on one XCD (4 M vertices and 16
    instances of the largest graph): every instance has the same parents, so
    the gradient of integer costs' sums is count times one instance's."""
    n = 65537
    rng = np.random.default_rng(count)
    src, dst, root = random_tree(rng, n, "random")
    G = sp.Graph(n, src, dst, np.ones(len(src), np.float32))
    arr = G.arrays()
    off, hd = arr["out_off"].cpu().numpy(), arr["out_dst"].cpu().numpy()
    pred = tree_pred(rng, n, off, hd, root, False)
    gc = rng.integers(-4, 5, n).astype(np.float32)  # exact in float32 throughout
    one = np.zeros(G.m, np.float32)
    tree_grad(n, off, hd, root, pred, gc, one)
    p = torch.from_numpy(pred).cuda().repeat(count)
    got = sp.backward([G], [0] * count, [root] * count, p, torch.from_numpy(gc).cuda().repeat(count))
    assert np.array_equal(got.cpu().numpy(), count * one)


def test_walk_on_xcds_matches_the_sweep(sp):
    """Instances of different sizes, roots, parents (some spoiled) and gradients,
    each on one XCD, against the same instances graph by graph, whose totals
    take the other walk (checked against ordered sums above)."""
    rng = np.random.default_rng(17)
    graphs = []
    for n, k in ((1, 0), (2, 5), (63, 300), (64, 200), (65, 400), (4097, 9000), (30011, 90000),
                 (60001, 200000)):
        src, dst = rng.integers(0, n, (2, k)).astype(np.int32)
        graphs.append(sp.Graph(n, src, dst, (0.5 + rng.random(k)).astype(np.float32)))
    inst = np.repeat(np.arange(8), [30, 30, 60, 60, 60, 150, 62, 33])
    rng.shuffle(inst)
    sources = [int(rng.integers(0, graphs[g].n)) for g in inst]
    sizes = np.array([graphs[g].n for g in inst])
    total = int(sizes.sum())
    assert total >= 1 << 22 and 16 * sizes.max() <= total
    _, pred, _ = sp.solve_batch(graphs, inst.tolist(), sources)
    bases = np.concatenate([[0], np.cumsum(sizes)])
    for i in range(0, len(inst), 40):  # any edge of the graph, mostly another vertex's
        g = graphs[inst[i]]
        at = torch.from_numpy(bases[i] + rng.integers(0, g.n, 1 + g.n // 50)).cuda()
        pred[at] = torch.from_numpy(rng.integers(-1, g.m + 1, len(at)).astype(np.int32)).cuda()
    gc = torch.randn(total, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    got = sp.backward(graphs, inst.tolist(), sources, pred, gc)
    part = 0
    for k, g in enumerate(graphs):
        mine = np.nonzero(inst == k)[0]
        cut = torch.cat([torch.arange(bases[i], bases[i + 1]) for i in mine]).cuda()
        assert len(cut) < 1 << 22
        want = sp.backward([g], [0] * len(mine), [sources[i] for i in mine], pred[cut], gc[cut])
        assert torch.equal(got[part:part + g.m], want), (k, g.n)
        part += g.m


@pytest.mark.parametrize("count", [7, 8, 9, 255, 256, 257, 513])
def test_gradient_over_many_instances(sp, count):
    """Around the instances that the gradient pass reads together and those it
    keeps the places of, vertices of few and of many in-edges."""
    rng = np.random.default_rng(count)
    n = 37
    src, dst, root = random_tree(rng, n, "star")
    G = sp.Graph(n, src, dst, rng.integers(1, 9, len(src)).astype(np.float32))
    arr = G.arrays()
    off, hd = arr["out_off"].cpu().numpy(), arr["out_dst"].cpu().numpy()
    want, preds, gcosts, sources = np.zeros(G.m, np.float32), [], [], []
    for i in range(count):
        r = root if i % 3 else int(rng.integers(0, n))
        pred = tree_pred(rng, n, off, hd, r, i % 5 == 0)
        gc = rng.standard_normal(n).astype(np.float32)
        tree_grad(n, off, hd, r, pred, gc, want)
        sources.append(r)
        preds.append(pred)
        gcosts.append(gc)
    got = sp.backward([G], [0] * count, sources, torch.from_numpy(np.concatenate(preds)).cuda(),
                      torch.from_numpy(np.concatenate(gcosts)).cuda())
    assert np.array_equal(got.cpu().numpy(), want)
