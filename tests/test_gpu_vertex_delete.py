"""Vertex deletes from a single id to all of them, so that the pass over the
pool stages from no slot to more than it holds (4096 of a workgroup's 8192),
and tails from one slot to more than a lane takes; ids repeated, past the table
and inactive.  Compared with the oracle, then the ids come back."""
import numpy as np
import pytest

from gpu_helpers import assert_same, need_gpu, say
from oracle import pyoracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 2, 4, 16])
@pytest.mark.parametrize("share", [0.0, 0.002, 0.03, 0.3, 0.75, 1.0])
def test_shares(B, share):
    gv = need_gpu()
    say(f"vertex delete: block {B}, share {share}")
    n = 4096
    rng = np.random.default_rng(int(share * 1000) + B)
    # degrees from none to some hundreds
    deg = (rng.pareto(1.2, n) * 20).astype(np.int64).clip(0, 600)
    deg[:4] = 0, 1, 16, 600
    s = np.repeat(np.arange(n), deg).astype(np.uint32)
    d = rng.integers(0, n, len(s)).astype(np.uint32)
    g = gv.Graph(n, s, d, block_slots=B)
    o = O.OracleGraph(n, s, d, block_slots=B)
    for r in range(2):
        ids = rng.choice(n, max(1, int(share * n)), replace=False).astype(np.uint32)
        ids = np.concatenate([ids, ids[: len(ids) // 3], rng.integers(n, 2 * n, 5)]).astype(np.uint32)
        ids = rng.permutation(ids)
        assert g.delete_vertices(ids) == o.delete_vertices(ids)[1], r
        assert_same(g, o, f"delete {r}")
        back = ids[ids < n][::2]
        assert g.insert_vertices(back) == o.insert_vertices(back)[1], r
        p = rng.integers(0, len(s), 2000)
        assert g.insert_edges(s[p], d[p]) == o.insert_edges(s[p], d[p])[1], r
        assert_same(g, o, f"insert {r}")
    g.close()
