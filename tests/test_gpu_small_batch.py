"""Batches whose graphs are all small: each instance in a workgroup of its own
with its state in LDS, against the oracle and against the persistent kernel
(small_n = -1), at the edges of the slot counts and of the register edges."""
import numpy as np
import pytest
import torch

import gen
from gpu_util import assert_same_solution, oracle_solution, sync, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sp():
    import paper_1812_10499_amd as sp
    assert torch.cuda.is_available()
    return sp


def rand_graph(rng, n, m, f32):
    src = rng.integers(0, n, m).astype(np.int32)
    dst = rng.integers(0, n, m).astype(np.int32)
    w = (rng.integers(1, 2**24, m) * 2.0 ** -24).astype(np.float32) if f32 else \
        rng.integers(1, 60, m).astype(np.int32)
    return gen.Graph("r", n, src, dst, w, 0)


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("sizes", [(1, 2, 1023, 1024), (1025, 7, 2048), (2049, 4095, 300), (4096,)])
def test_small_batch(sp, f32, sizes):
    rng = np.random.default_rng(sum(sizes))
    glist, graphs = [], []
    for k, n in enumerate(sizes):
        g = rand_graph(rng, n, int(n * (2 + 3 * k)), f32)
        glist.append(g)
        graphs.append(sp.Graph(g.n, g.src, g.dst, g.w, order=("degree" if k % 2 else "input"),
                               scope=("open", "all", "auto")[k % 3],
                               relax=("setting", "correcting")[(k + f32) % 2]))
    inst = [i % len(sizes) for i in range(2 * len(sizes) + 1)]
    srcs = [int(rng.integers(0, glist[g].n)) for g in inst]
    print("small batch", sizes, f32, flush=True)
    out = {}
    for name, launch in (("lds", None), ("grid", dict(small_n=-1, wg=-1))):
        sp.set_launch(launch)
        try:
            cost, pred, st = sp.solve_batch(graphs, inst, srcs, with_pred=True, with_stats=True)
            c2, none, _ = sp.solve_batch(graphs, inst, srcs, with_pred=False)
            sync()
            assert none is None and torch.equal(c2, cost)
        finally:
            sp.set_launch(None)
        out[name] = (to_np(cost), to_np(pred), st)
    assert np.array_equal(out["lds"][0], out["grid"][0])
    assert np.array_equal(out["lds"][1], out["grid"][1])
    assert out["lds"][2] == out["grid"][2]
    base = 0
    for i, (gi, s) in enumerate(zip(inst, srcs)):
        g = glist[gi]
        ref = oracle_solution(g.n, g.src, g.dst, g.w, s, graphs[gi].effective_scope,
                              graphs[gi].effective_relax, graphs[gi].effective_delta)
        assert_same_solution(torch.from_numpy(out["lds"][0][base:base + g.n]),
                             torch.from_numpy(out["lds"][1][base:base + g.n]),
                             out["lds"][2][i], ref, "inst %d" % i)
        base += g.n


def test_small_batch_hubs_and_ties(sp):
    # out-lists and in-lists of a thousand edges, and float32 edges below half
    # an ulp of the cost (the equal-cost rule in several instances at once)
    n = 1500
    star = np.arange(1, n, dtype=np.int32)
    zero = np.zeros(n - 1, np.int32)
    src = np.concatenate([zero, star]).astype(np.int32)
    dst = np.concatenate([star, zero]).astype(np.int32)
    w = (1 + np.arange(len(src)) % 97).astype(np.float32)
    chain = gen.Graph("ties", 40, np.arange(39, dtype=np.int32), np.arange(1, 40, dtype=np.int32),
                      np.array([1.0] + [2.0 ** -30] * 38, np.float32), 0)
    glist = [gen.Graph("star", n, src, dst, w, 0), chain]
    graphs = [sp.Graph(g.n, g.src, g.dst, g.w) for g in glist]
    inst, srcs = [1, 0, 1, 0, 1], [0, 3, 0, 0, 5]
    cost, pred, st = sp.solve_batch(graphs, inst, srcs, with_pred=True, with_stats=True)
    sync()
    base = 0
    for i, (gi, s) in enumerate(zip(inst, srcs)):
        g = glist[gi]
        ref = oracle_solution(g.n, g.src, g.dst, g.w, s, graphs[gi].effective_scope,
                              graphs[gi].effective_relax, graphs[gi].effective_delta)
        assert_same_solution(cost[base:base + g.n], pred[base:base + g.n], st[i], ref, "%d" % i)
        base += g.n
    sp.check()


def test_small_batch_watchdog(sp):
    # a limit of one round: every instance ends with the fault status
    g = gen.random_workload(n=600, m=4000)
    G = sp.Graph(g.n, g.src, g.dst, g.w)
    sp.set_round_limit(1)
    try:
        with pytest.raises(sp.SSSPError):
            sp.solve_batch([G], [0, 0, 0], [0, 1, 2], with_stats=True)
        sp.solve_batch([G], [0, 0], [0, 1])
        with pytest.raises(sp.SSSPError):
            sp.check()
    finally:
        sp.set_round_limit(0)
    cost, _, _ = sp.solve_batch([G], [0, 0], [0, 0])
    sp.check()
    assert torch.equal(cost[:g.n], cost[g.n:])


@pytest.mark.parametrize("n", [1000, 2011, 4090])
def test_long_out_lists(sp, n):
    # out-degrees around the lines between 8 lanes, a wave and the whole block
    # to an out-list, several of each in one relax set
    rng = np.random.default_rng(n)
    degs = [1, 7, 8, 9, 63, 64, 65, 127, 256, 257, 1023, 1024, 1025, 1100, 2500]
    tails = rng.permutation(n)[:3 * len(degs)]
    src = [np.zeros(len(tails), np.int64), np.repeat(tails, np.tile(degs, 3))]
    dst = [tails, rng.integers(0, n, 3 * sum(degs))]
    src += [rng.integers(0, n, 2 * n)]
    dst += [rng.integers(0, n, 2 * n)]
    src, dst = np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32)
    w = rng.integers(1, 4, len(src)).astype(np.int32)
    for scope, relax in (("open", "setting"), ("all", "correcting")):
        G = sp.Graph(n, src, dst, w, scope=scope, relax=relax)
        ref = oracle_solution(n, src, dst, w, 0, scope, G.effective_relax, G.effective_delta)
        print("long lists", n, scope, relax, flush=True)
        cost, pred, st = sp.solve(G, 0, with_stats=True)
        bc, bp, bst = sp.solve_batch([G], [0, 0], [0, int(tails[-1])], with_stats=True)
        sync()
        assert_same_solution(cost, pred, st, ref, "single")
        assert_same_solution(bc[:n], bp[:n], bst[0], ref, "batch")
