"""A plan recorded on a graph that has run nothing yet: every buffer of its
runs is sized before the recording, for the deletes of a coalesced run as for
its inserts."""
import numpy as np
import pytest

from gpu_helpers import assert_same, need_gpu, say
from oracle import pyoracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [1, 64, 3000, 9000, 40000, 300000])
@pytest.mark.parametrize("coalesce", [0, 1])
@pytest.mark.parametrize("overlap", [0, 1])
def test_recorded_first(size, coalesce, overlap):
    gv = need_gpu()
    say(f"plan on a fresh graph: {size} pairs, coalesce {coalesce}, overlap {overlap}")
    n = 1 << 13
    rng = np.random.default_rng(size)
    s, d = (rng.integers(0, n, size).astype(np.uint32) for _ in range(2))
    g = gv.Graph(n, s[: size // 2], d[: size // 2], block_slots=8)
    o = O.OracleGraph(n, s[: size // 2], d[: size // 2], block_slots=8)
    gv.gv_set_tuning(g.h, coalesce=coalesce, overlap=overlap)
    half = size // 2
    ops = [(1, s[:half + 1], d[:half + 1]), (0, s, d), (1, s[half // 2:], d[half // 2:])]
    plan = gv.Plan(g.h, ops)
    for _ in range(3):
        plan.launch()
        for kind, a, b in ops:
            (o.insert_edges if kind == 0 else o.delete_edges)(a, b)
        g.sync()
        assert_same(g, o)
    plan.close()
    g.close()
