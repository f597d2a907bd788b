"""Teams of single-wave workgroups (the default for few instances on graphs of
low degree spread under C scope OPEN) against the oracle, the one-workgroup
kernel (wg = 1) and, where a team's room runs out, the second run."""
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


def regular(rng, n, k, f32=False):
    """Every vertex has k out- and k in-edges: low degree spread, and a
    wavefront of most of the graph."""
    src = np.repeat(np.arange(n, dtype=np.int32), k)
    dst = np.concatenate([rng.permutation(n) for _ in range(k)]).reshape(k, n).T.reshape(-1)
    w = (rng.integers(1, 2**24, n * k) * 2.0 ** -24).astype(np.float32) if f32 else \
        rng.integers(1, 50, n * k).astype(np.int32)
    return gen.Graph("regular", n, src, dst.astype(np.int32), w, 3)


def rect(rows, cols, w):
    src, dst = gen.grid_edges(rows, cols)
    return gen.Graph("rect", rows * cols, src, dst, w(len(src)), (rows * cols) // 3)


def three_ways(sp, g, label, **kw):
    G = sp.Graph(g.n, g.src, g.dst, g.w, scope="open", **kw)
    assert G.kernel == "wg_rounds_kernel", G.policy()
    ref = oracle_solution(g.n, g.src, g.dst, g.w, g.source, "open", G.effective_relax,
                          G.effective_delta)
    print("mesh", label, g.n, ref["rounds"], flush=True)
    for launch in (None, dict(wg=1), dict(blocks=2)):
        sp.set_launch(launch)
        try:
            cost, pred, st = sp.solve(G, g.source, with_stats=True)
            sync()
        finally:
            sp.set_launch(None)
        assert_same_solution(cost, pred, st, ref, "%s %s" % (label, launch))
    sp.check()
    return G, ref


# sizes around the team sizes' lines (512 vertices a wave), 1 x n strips, and
# both relax steps (wide and narrow weights)
@pytest.mark.parametrize("rows,cols,whi", [(65, 64, 1000), (64, 65, 1), (1, 5000, 7), (90, 91, 9),
                                           (128, 127, 1000), (255, 129, 20), (40, 1600, 1000)])
def test_grids(sp, rows, cols, whi):
    rng = np.random.default_rng(rows)
    three_ways(sp, rect(rows, cols, lambda m: rng.integers(1, whi + 1, m).astype(np.int32)),
               "%dx%d" % (rows, cols))


@pytest.mark.parametrize("order", ["input", "degree"])
def test_float_grid(sp, order):
    rng = np.random.default_rng(5)
    three_ways(sp, rect(70, 75, lambda m: (0.5 + rng.random(m)).astype(np.float32)), "f32",
               order=order)


def test_tiny_float_weights(sp):
    # below half an ulp of the cost: the equal-cost rule behind the team
    rng = np.random.default_rng(6)
    three_ways(sp, rect(67, 70, lambda m: np.where(rng.random(m) < 0.4, 2.0 ** -40, 1.0)
                        .astype(np.float32)), "ties")


@pytest.mark.parametrize("k,f32", [(5, False), (9, True)])
def test_room_runs_out(sp, k, f32):
    # the open set outgrows the seats (or the mailboxes): run again in one
    # workgroup; in-lists longer than the seats' register edges
    three_ways(sp, regular(np.random.default_rng(k), 20000, k, f32), "regular%d" % k)


# Open sets that no team holds, by counting alone: more open vertices a round, in
# the mean, than 64 waves of 256 seats; or more first discoveries in round 2 than
# the mailboxes of a team of two waves (blocks = 2) take, 16 from each to each.
@pytest.mark.parametrize("kind,f32,kw", [
    ("seats", False, dict()), ("seats", True, dict(order="degree")),
    ("seats", False, dict(relax="correcting")), ("seats", False, dict(relax="correcting", delta=9)),
    ("boxes", False, dict()), ("boxes", True, dict(relax="correcting"))])
def test_goes_on_in_one_workgroup(sp, kind, f32, kw):
    rng = np.random.default_rng(11)
    if kind == "seats":
        g = regular(rng, 160000, 7, f32)
    else:
        g = regular(rng, 5000, 16, f32)
        g.w[:] = 1
    G, ref = three_ways(sp, g, "outgrown %s" % kind, **kw)
    if kind == "seats":
        assert ref["open_visits"] > 64 * 256 * ref["rounds"]
    else:
        # unit weights: round 1 fixes the source's neighbours, round 2 discovers
        # theirs
        first = np.unique(g.dst[g.src == g.source])
        second = np.unique(g.dst[np.isin(g.src, first)])
        assert len(np.setdiff1d(second, np.append(first, g.source))) > 2 * 2 * 16
    # the rounds run by both kernels stop at a target as those of one do
    order = np.argsort(ref["cost"], kind="stable")
    for t in (int(order[1]), int(order[g.n // 2]), int(order[-1])):
        out = []
        for launch in (None, dict(wg=1)):
            sp.set_launch(launch)
            try:
                c, st = sp.solve_target(G, g.source, t, with_stats=True)
                sync()
            finally:
                sp.set_launch(None)
            out.append((to_np(c), st))
        assert np.array_equal(out[0][0], out[1][0]) and out[0][1] == out[1][1], t


def test_profile_covers_both_kernels(sp):
    # what the profiler reports of a solve that outgrew its team includes the
    # rounds behind the team: no less than most of the one workgroup's time
    g = regular(np.random.default_rng(12), 90000, 6)
    G = sp.Graph(g.n, g.src, g.dst, g.w, scope="open")
    ms = {}
    for name, launch in (("team", None), ("one", dict(wg=1))):
        sp.set_launch(launch)
        try:
            sp.solve(G, g.source)
            sync()
            sp.sssp_profile_read()
            sp.sssp_profile_enable(True)
            for _ in range(3):
                sp.solve(G, g.source)
            sync()
            launches, ms[name] = sp.sssp_profile_read()
        finally:
            sp.sssp_profile_enable(False)
            sp.set_launch(None)
        assert launches == 3
    print("profile", ms, flush=True)
    assert ms["team"] > 0.5 * ms["one"]


def test_target(sp):
    g = gen.grid_workload(side=80)
    G, ref = three_ways(sp, g, "target")
    order = np.argsort(ref["cost"], kind="stable")
    for t in (g.source, int(order[1]), int(order[g.n // 2]), int(order[-1])):
        out = []
        for launch in (None, dict(wg=1)):
            sp.set_launch(launch)
            try:
                c, st = sp.solve_target(G, g.source, t, with_stats=True)
                sync()
            finally:
                sp.set_launch(None)
            out.append((to_np(c), st))
        assert np.array_equal(out[0][0], out[1][0]) and out[0][1] == out[1][1], t
        assert out[0][0][t] == ref["cost"][t]


@pytest.mark.parametrize("count", [1, 8, 9, 128, 129])
def test_batches(sp, count):
    # teams of one launch on several graphs, one of which gives up; 129
    # instances are one more than teams are used for
    rng = np.random.default_rng(count)
    glist = [rect(66, 66, lambda m: (0.5 + rng.random(m)).astype(np.float32)),
             rect(50, 130, lambda m: (rng.integers(1, 2**24, m) * 2.0 ** -24).astype(np.float32)),
             regular(rng, 9000, 7, True)]
    graphs = [sp.Graph(g.n, g.src, g.dst, g.w, scope="open") for g in glist]
    inst = [i % 3 for i in range(count)]
    srcs = [int(rng.integers(0, glist[g].n)) for g in inst]
    out = []
    for launch in (None, dict(wg=1)):
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
    for _ in range(3):  # replays, with eager work and a synchronization between
        plan.run()
        sp.solve(graphs[0], 1)
        sync()
        assert np.array_equal(to_np(plan.cost), out[0][0])
        assert np.array_equal(to_np(plan.pred), out[0][1])
        assert plan.stats() == out[0][2]
    plan.close()


def test_watchdog(sp):
    g = gen.grid_workload(side=70)
    G = sp.Graph(g.n, g.src, g.dst, g.w)
    sp.set_round_limit(5)
    try:
        with pytest.raises(sp.SSSPError):
            sp.solve(G, g.source, with_stats=True)
    finally:
        sp.set_round_limit(0)
    with pytest.raises(sp.SSSPError):
        sp.check()
    sp.solve(G, g.source)
    sp.check()
