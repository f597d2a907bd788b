"""Teams that own every vertex (the default under C scope ALL without hubs)
against the oracle and the grid-wide kernel (wg = -1)."""
import numpy as np
import pytest
import torch

import gen
import oracle
from gpu_util import assert_same_solution, oracle_solution, sync, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sp():
    import paper_1812_10499_amd as sp
    assert torch.cuda.is_available()
    return sp


def rand(rng, n, m, kind):
    src = rng.integers(0, n, m).astype(np.int32)
    dst = rng.integers(0, n, m).astype(np.int32)
    if kind == "f32":
        w = (rng.integers(1, 2**24, m) * 2.0 ** -24).astype(np.float32)
    elif kind == "ties":  # mostly below half an ulp of the cost
        w = np.where(rng.random(m) < 0.8, 2.0 ** -40, 1.0).astype(np.float32)
    else:
        w = rng.integers(1, 1 + kind, m).astype(np.int32)
    return gen.Graph("rand", n, src, dst, w, int(rng.integers(0, n)))


def both(sp, g, label, launches=(None, dict(wg=-1)), **kw):
    G = sp.Graph(g.n, g.src, g.dst, g.w, scope="all", **kw)
    ref = oracle_solution(g.n, g.src, g.dst, g.w, g.source, "all", G.effective_relax,
                          G.effective_delta)
    print("dense", label, g.n, g.m, ref["rounds"], ref["settles"], flush=True)
    for launch in launches:
        sp.set_launch(launch)
        try:
            cost, pred, st = sp.solve(G, g.source, with_stats=True)
            sync()
        finally:
            sp.set_launch(None)
        assert_same_solution(cost, pred, st, ref, "%s %s" % (label, launch))
    sp.check()
    return G, ref


# around one block's vertices, several blocks, the line to one team over all
# XCDs; unit weights; sparse graphs, mostly unreachable
@pytest.mark.parametrize("n,deg,kind", [
    (4097, 8, 100), (5119, 3, "f32"), (8193, 8, 1), (20011, 2, 100), (32768, 7, "f32"),
    (36864, 5, 30), (36865, 5, 30), (50001, 1, 9), (100003, 6, "f32"), (262145, 4, 1)])
def test_random(sp, n, deg, kind):
    both(sp, rand(np.random.default_rng(n), n, n * deg, kind), "random")


@pytest.mark.parametrize("n", [6000, 40000])
@pytest.mark.parametrize("kind,kw", [
    (100, dict(relax="correcting")), (1000, dict(relax="correcting", delta=200)),
    ("f32", dict(relax="correcting", order="degree")), ("ties", dict()),
    ("ties", dict(relax="correcting"))])
def test_modes(sp, n, kind, kw):
    both(sp, rand(np.random.default_rng(7), n, 5 * n, kind), "modes", **kw)


def test_few_blocks(sp):
    # a grid limited to 16 blocks (teams of two), and to 4 (the grid-wide kernel)
    both(sp, rand(np.random.default_rng(9), 30000, 150000, 20), "few",
         launches=(dict(blocks=16), dict(blocks=4)))


def test_degree_line(sp):
    # a vertex of 256 and of 257 edges: the line to the grid-wide kernel
    for hub in (254, 255, 256):
        rng = np.random.default_rng(hub)
        g = rand(rng, 9000, 20000, 50)
        keep = (g.src != 5) & (g.dst != 5)
        extra = rng.integers(6, 9000, hub).astype(np.int32)
        src = np.concatenate([g.src[keep], np.full(hub, 5, np.int32), [0]]).astype(np.int32)
        dst = np.concatenate([g.dst[keep], extra, [5]]).astype(np.int32)
        w = rng.integers(1, 50, len(src)).astype(np.int32)
        both(sp, gen.Graph("hub", 9000, src, dst, w, 0), "hub%d" % hub)


@pytest.mark.parametrize("n", [7000, 60000])
def test_target(sp, n):
    g = rand(np.random.default_rng(n), n, 6 * n, 100)
    G, ref = both(sp, g, "target")
    order = np.argsort(ref["cost"], kind="stable")
    for t in (g.source, int(order[1]), int(order[n // 2]), int(order[-1])):
        out = []
        for launch in (None, dict(wg=-1)):
            sp.set_launch(launch)
            try:
                c, st = sp.solve_target(G, g.source, t, with_stats=True)
                sync()
            finally:
                sp.set_launch(None)
            out.append((to_np(c), st))
        assert np.array_equal(out[0][0], out[1][0]) and out[0][1] == out[1][1], t


@pytest.mark.parametrize("count,lo,hi,kind", [(2, 5000, 9000, 50), (40, 29000, 30000, 1),
                                              (70, 4000, 9000, "f32"), (300, 100, 5000, 12)])
def test_batches(sp, count, lo, hi, kind):
    # queues of instances; with unit weights and four blocks to a team a
    # round fixes more vertices than a block's LDS list holds
    rng = np.random.default_rng(count)
    glist = [rand(rng, int(rng.integers(lo, hi)), 0, 1) for _ in range(min(count, 12))]
    glist = [rand(rng, g.n, int(g.n * rng.integers(3, 9)), kind) for g in glist]
    graphs = [sp.Graph(g.n, g.src, g.dst, g.w, scope="all",
                       relax=("correcting" if k % 3 == 1 else "setting"))
              for k, g in enumerate(glist)]
    inst = [int(rng.integers(0, len(glist))) for _ in range(count)]
    srcs = [int(rng.integers(0, glist[g].n)) for g in inst]
    print("dense batch", count, lo, hi, kind, flush=True)
    out = []
    for launch in (dict(small_n=-1), dict(small_n=-1, wg=-1)):
        sp.set_launch(launch)
        try:
            c, p, st = sp.solve_batch(graphs, inst, srcs, with_stats=True)
            c2, _, _ = sp.solve_batch(graphs, inst, srcs, with_pred=False)
            sync()
            assert torch.equal(c, c2)
        finally:
            sp.set_launch(None)
        out.append((to_np(c), to_np(p), st))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    assert out[0][2] == out[1][2]
    plan = sp.Plan(graphs, inst, srcs, with_stats=True, launch=dict(small_n=-1))
    for _ in range(3):  # replays, with eager work and a synchronization between
        plan.run()
        sp.solve(graphs[0], 0)
        sync()
        assert np.array_equal(to_np(plan.cost), out[0][0])
        assert plan.stats() == out[0][2]
    plan.close()
    bases, _ = sp.batch_layout(graphs, inst)
    for i in (0, count - 1):
        g = glist[inst[i]]
        ref = oracle_solution(g.n, g.src, g.dst, g.w, srcs[i], "all",
                              graphs[inst[i]].effective_relax, graphs[inst[i]].effective_delta)
        sl = slice(bases[i], bases[i] + g.n)
        assert_same_solution(torch.from_numpy(out[0][0][sl]), torch.from_numpy(out[0][1][sl]),
                             out[0][2][i], ref, "inst %d" % i)


@pytest.mark.parametrize("n,kind,relax", [
    (36864, 100, "setting"), (36865, 100, "setting"), (40001, "f32", "correcting"),
    (40001, 100, "correcting"), (150001, 50, "setting"), (150001, "f32", "setting")])
def test_batch_of_one(sp, n, kind, relax):
    # one instance may be a team over all XCDs, whose every block has to be
    # waited for and heard, in a batch and a plan as in a single solve; also
    # with fewer blocks than a wave has lanes, and not a multiple of them
    g = rand(np.random.default_rng(n), n, 8 * n, kind)
    G = sp.Graph(g.n, g.src, g.dst, g.w, scope="all", relax=relax)
    ref = oracle_solution(g.n, g.src, g.dst, g.w, g.source, "all", G.effective_relax,
                          G.effective_delta)
    for launch in (None, dict(blocks=16), dict(blocks=100)):
        print("dense one", n, kind, relax, launch, flush=True)
        sp.set_launch(launch)
        try:
            out = sp.solve(G, g.source, with_stats=True)
            cost, pred, st = sp.solve_batch([G], [0], [g.source], with_stats=True)
            sync()
        finally:
            sp.set_launch(None)
        assert_same_solution(*out, ref, "single %s" % launch)
        assert_same_solution(cost, pred, st[0], ref, "batch %s" % launch)
    plan = sp.Plan([G], [0], [g.source], with_stats=True)
    for _ in range(3):  # replays, with eager work and a synchronization between
        plan.cost.zero_()
        plan.run()
        sync()
        assert_same_solution(plan.cost, plan.pred, plan.stats()[0], ref, "plan")
    plan.close()
    sp.check()


@pytest.mark.parametrize("where", [0, 33, 69])
def test_mixed_sizes(sp, where):
    # a queue of small instances (1 vertex upwards) with a large one among them,
    # which is taken first wherever it stands
    rng = np.random.default_rng(where)
    sizes = [1, 2, 7, 8, 9, 15, 16, 100, 127, 129, 500, 1000, 5000]
    glist = [rand(rng, n, 6 * n, 40) for n in sizes] + [rand(rng, 70001, 6 * 70001, 40)]
    graphs = [sp.Graph(g.n, g.src, g.dst, g.w, scope="all") for g in glist]
    inst = [i % len(sizes) for i in range(69)]
    inst.insert(where, len(sizes))
    srcs = [int(rng.integers(0, glist[g].n)) for g in inst]
    print("dense mixed", where, flush=True)
    out = []
    for launch in (None, dict(wg=-1)):
        sp.set_launch(launch)
        try:
            c, p, st = sp.solve_batch(graphs, inst, srcs, with_stats=True)
            sync()
        finally:
            sp.set_launch(None)
        out.append((to_np(c), to_np(p), st))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    assert out[0][2] == out[1][2]
    plan = sp.Plan(graphs, inst, srcs, with_stats=True)
    plan.run()
    sync()
    assert np.array_equal(to_np(plan.cost), out[0][0]) and plan.stats() == out[0][2]
    plan.close()


@pytest.mark.parametrize("sizes,kind", [((163840, 900), 20), ((163841, 5, 163000), 20),
                                        ((5, 163841), "f32"), ((7000, 491521, 40000), 9)])
def test_few_large_instances(sp, sizes, kind):
    # two or three instances, around the lines from which they share a team over
    # all XCDs
    rng = np.random.default_rng(sizes[0])
    glist = [rand(rng, n, 4 * n, kind) for n in sizes]
    graphs = [sp.Graph(g.n, g.src, g.dst, g.w, scope="all",
                       relax=("correcting" if k == 1 else "setting"))
              for k, g in enumerate(glist)]
    which, srcs = list(range(len(sizes))), [g.source for g in glist]
    print("dense few", sizes, kind, flush=True)
    cost, pred, st = sp.solve_batch(graphs, which, srcs, with_stats=True)
    sync()
    bases, _ = sp.batch_layout(graphs, which)
    plan = sp.Plan(graphs, which, srcs, with_stats=True)
    for _ in range(2):
        plan.run()
        sp.solve(graphs[0], 0)
        sync()
        assert torch.equal(plan.cost, cost) and torch.equal(plan.pred, pred)
        assert plan.stats() == st
    plan.close()
    for k, g in enumerate(glist):
        ref = oracle_solution(g.n, g.src, g.dst, g.w, g.source, "all",
                              graphs[k].effective_relax, graphs[k].effective_delta)
        sl = slice(bases[k], bases[k] + g.n)
        assert_same_solution(cost[sl], pred[sl], st[k], ref, "inst %d" % k)
    sp.check()


def test_training_step_of_one_source(sp):
    n = 40001
    g = rand(np.random.default_rng(3), n, 8 * n, "f32")
    G = sp.Graph(g.n, g.src, g.dst, g.w)
    assert G.effective_scope == "all"
    w = torch.from_numpy(g.w).cuda().requires_grad_()
    ref = oracle_solution(g.n, g.src, g.dst, g.w, g.source)
    cost = sp.shortest_paths(w, G, [g.source], order="coo")
    (gw,) = torch.autograd.grad(cost.sum(), w)
    assert np.array_equal(to_np(cost)[0], ref["cost"])
    # unit coefficients: whole numbers, exact in any order
    want = oracle.grad(ref["csr"], [g.source], ref["pred"].reshape(1, n), np.ones((1, n)))
    assert np.array_equal(to_np(gw)[to_np(G.perm)].astype(np.float64), want)


def test_watchdog(sp):
    for n in (6000, 50000):
        g = gen.random_workload(n=n, m=6 * n)
        G = sp.Graph(g.n, g.src, g.dst, g.w, scope="all")
        sp.set_round_limit(3)
        try:
            with pytest.raises(sp.SSSPError):
                sp.solve(G, g.source, with_stats=True)
            with pytest.raises(sp.SSSPError):
                sp.solve_batch([G], [0, 0, 0], [0, 1, 2], with_stats=True)
        finally:
            sp.set_round_limit(0)
        with pytest.raises(sp.SSSPError):
            sp.check()
        sp.solve(G, g.source)
        sp.check()
