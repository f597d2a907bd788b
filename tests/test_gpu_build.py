"""The builder's sorts where they can go wrong: tile edges, digit widths,
both tile sizes, the longest lists of the rank sort and of the lane groups."""
import numpy as np
import pytest
import torch

from gpu_util import check_solver_copy, sync, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sp():
    import paper_1812_10499_amd as sp
    assert torch.cuda.is_available()
    return sp


def weights(rng, kind, m):
    if kind == "f32":
        return (rng.integers(1, 2**24, m) * 2.0 ** -24).astype(np.float32)
    return rng.integers(1, 1 + kind, m).astype(np.int32)


@pytest.mark.parametrize("n,m,order,kind", [
    (1, 1, "input", 3), (2, 4095, "degree", 1), (2049, 4096, "auto", "f32"),
    (2048, 4097, "degree", "f32"), (70000, 65537, "input", 2000), (70000, 65535, "degree", 30000),
    (4194305, 9000, "degree", 5), (5, 0, "degree", 1), (300, 40000, "input", "f32"),
    (9000, 4194304 + 17, "degree", 2047), (100000, 4194304 - 1, "input", "f32"),
])
def test_build_and_reweight(sp, n, m, order, kind):
    print("build", n, m, order, kind, flush=True)
    rng = np.random.default_rng(n + m)
    src = rng.integers(0, n, m).astype(np.int32)
    dst = rng.integers(0, n, m).astype(np.int32)
    w = weights(rng, kind, m)
    G = sp.Graph(n, src, dst, w, order=order)
    sync()
    check_solver_copy(G, n, src, dst, w)
    if m:
        w2 = weights(rng, kind, m)
        G.set_weights(G.to_edge_order(torch.from_numpy(w2).cuda()))
        sync()
        check_solver_copy(G, n, src, dst, w2)


@pytest.mark.parametrize("length", [8, 127, 128, 129, 1024, 1025, 3000])
@pytest.mark.parametrize("side", ["in", "out"])
def test_one_long_list(sp, side, length):
    # one vertex with `length` in- or out-edges of equal and unequal weights
    # among lists of 0 to 2 entries
    rng = np.random.default_rng(length)
    n = 5000
    a = np.full(length, 1234, np.int32)
    b = rng.integers(0, n, length).astype(np.int32)
    s2, d2 = rng.integers(0, n, 4000).astype(np.int32), rng.integers(0, n, 4000).astype(np.int32)
    src = np.concatenate([s2, a if side == "out" else b])
    dst = np.concatenate([d2, b if side == "out" else a])
    p = rng.permutation(len(src))
    src, dst = src[p], dst[p]
    w = rng.integers(1, 40, len(src)).astype(np.int32)
    for order in ("input", "degree"):
        G = sp.Graph(n, src, dst, w, order=order)
        sync()
        check_solver_copy(G, n, src, dst, w)


def test_bad_edges_and_weights_refused(sp):
    # endpoints are checked after the sorts have run over them
    w = np.array([1, 2, 3], np.int32)
    for src, dst in (([0, 5, 1], [1, 2, 3]), ([0, 1, 2], [1, -1, 3]),
                     ([0, 1, 2**31 - 1], [1, 2, 3])):
        with pytest.raises(sp.SSSPError):
            sp.Graph(4, np.array(src, np.int32), np.array(dst, np.int32), w)
    with pytest.raises(sp.SSSPError):
        sp.Graph(4, np.array([0, 1, 2], np.int32), np.array([1, 2, 3], np.int32),
                 np.array([1, 0, 3], np.int32))
    G = sp.Graph(4, np.array([0, 1, 2], np.int32), np.array([1, 2, 3], np.int32), w)
    with pytest.raises(sp.SSSPError):
        G.set_weights(torch.tensor([1, -2, 3], dtype=torch.int32))
    sync()
    assert np.array_equal(to_np(G.arrays()["out_w"]), w)


@pytest.mark.parametrize("n,m", [(1000, 8000), (1000000, 8000001), (6000001, 900)])
def test_workspace(sp, n, m):
    # what a build and new weights take of the device beside the graph's own
    # buffer, from an empty workspace: 20 bytes an edge (16 a vertex where there
    # are more vertices), the digit counts and an eighth of headroom
    g = torch.Generator(device="cuda").manual_seed(n)
    src, dst = (torch.randint(0, n, (m,), generator=g, device="cuda", dtype=torch.int32)
                for _ in range(2))
    w = torch.rand(m, generator=g, device="cuda") + 0.5
    G = sp.Graph(n, src, dst, w, order="degree")  # (code objects, the allocator's pool)
    we = G.to_edge_order(w)
    want = {k: v.clone() for k, v in G.solver_arrays().items()}
    sync()
    sp.sssp_release_workspace()
    free = torch.cuda.mem_get_info()[0]
    held = torch.cuda.memory_reserved()
    del G
    G = sp.Graph(n, src, dst, w, order="degree")
    G.set_weights(we)
    sync()
    assert torch.cuda.memory_reserved() == held  # (the graph's buffer is the old one's)
    taken = free - torch.cuda.mem_get_info()[0]
    counts = (max(m, n) // 4096 + 2) * 2048 * 4
    most = 1.13 * (16 * max(m, n) + 4 * m + counts)
    print("workspace", n, m, taken, int(most), flush=True)
    assert taken <= most + (8 << 20)  # (allocations are whole pages of 2 MiB)
    for k, v in G.solver_arrays().items():
        assert torch.equal(v, want[k]), k
