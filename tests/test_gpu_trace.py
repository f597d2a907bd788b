"""The round trace (SSSP_TRACE): a row a round with its time stamps, and per-block
records of the blocks that the kernel ran, no others."""
import numpy as np
import pytest
import torch

import gen
from gpu_util import sync

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sp():
    import paper_1812_10499_amd as sp
    assert torch.cuda.is_available()
    return sp


@pytest.mark.parametrize("name,blocks", [("random", None), ("skewed", None), ("skewed", 40)])
def test_trace_rows(sp, tmp_path, monkeypatch, name, blocks):
    g = gen.random_workload(n=9000, m=72000) if name == "random" else gen.rmat_workload(scale=14)
    G = sp.Graph(g.n, g.src, g.dst, g.w)
    assert G.kernel == "rounds_kernel"
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    path = tmp_path / "trace"
    sp.set_launch(dict(blocks=blocks) if blocks else None)
    try:
        c0, _, st0 = sp.solve(G, g.source, with_stats=True)
        monkeypatch.setenv("SSSP_TRACE", str(path))
        c1, _, st1 = sp.solve(G, g.source, with_stats=True)
        sync()
    finally:
        monkeypatch.delenv("SSSP_TRACE", raising=False)
        sp.set_launch(None)
    assert torch.equal(c0, c1) and st0 == st1
    rows = [r.split(",") for r in path.read_text().splitlines()]
    assert rows[0][:2] == ["round", "start"] and len(rows) == 1 + st1["rounds"]
    start = [int(r[1]) for r in rows[1:]]
    assert min(start) > 0 and start == sorted(start)
    ef = rows[0].index("ef")
    assert sum(int(r[ef]) for r in rows[1:]) == st1["relaxed_edges"]
    blk = np.loadtxt(str(path) + ".blk", delimiter=",", dtype=np.int64)
    ran = blocks or cus // 2  # (half the grid for a graph of this size)
    assert blk[:, 2].max() == ran - 1 and (blk[blk[:, 2] == ran - 1, 3] > 0).any()
