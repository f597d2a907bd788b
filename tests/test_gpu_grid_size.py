"""The grid-wide kernel's default grid on both sides of the line at 6291456
edges (half of the compute units up to it) against the full grid, one block
and a grid that is no power of two: costs, parents and counters agree."""
import numpy as np
import pytest
import torch

from gpu_util import sync, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [6291456, 6291457])
def test_default_grid_by_edges(m):
    import paper_1812_10499_amd as sp
    assert torch.cuda.is_available()
    rng = np.random.default_rng(m)
    n = 700001
    src = rng.integers(0, n, m).astype(np.int32)
    src[: m // 3] = src[: m // 3] % 1000  # hubs: no team owns every vertex
    dst = rng.integers(0, n, m).astype(np.int32)
    G = sp.Graph(n, src, dst, rng.integers(1, 200, m).astype(np.int32))
    got = []
    full = torch.cuda.get_device_properties(0).multi_processor_count
    for launch in (None, dict(blocks=full), dict(blocks=7)):
        sp.set_launch(launch)
        try:
            cost, pred, st = sp.solve(G, 3, with_stats=True)
            sync()
        finally:
            sp.set_launch(None)
        got.append((to_np(cost), to_np(pred),
                    {k: v for k, v in st.items() if k not in ("ms", "solo_phases")}))
    for c, p, s in got[1:]:
        assert np.array_equal(c, got[0][0]) and np.array_equal(p, got[0][1]) and s == got[0][2]
