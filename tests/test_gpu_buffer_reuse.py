"""Graphs whose pool and scratch are buffers of a destroyed graph, with that
graph's slots, owner records, directory and marks in them."""
import numpy as np
import pytest

from gpu_helpers import assert_same, need_gpu, same_answers, say
from oracle import pyoracle as O

pytestmark = pytest.mark.gpu

N = 1 << 14
POOL = 64 << 20


def _pool_bytes(B):
    """A pool that takes, with its lists and attribute words, nearly as much
    memory as that of POOL bytes in blocks of 8: a block has 4 B per slot, as
    much for one attribute word, and 44 B of lists, owner and directory."""
    blocks = int(0.97 * (POOL // 32) * (8 * 8 + 44) / (8 * B + 44))
    return 4 * B * blocks


def _pairs(rng, size):
    return tuple(rng.integers(0, N, size).astype(np.uint32) for _ in range(2))


def _used_graph(gv):
    """A graph with longer adjacencies, grown and shrunk; its buffers are kept
    when it is closed."""
    rng = np.random.default_rng(1)
    s, d = _pairs(rng, 400000)
    g = gv.Graph(N, s, d, block_slots=8, pool_bytes=POOL, edge_attr_words=1)
    g.set_edge_attrs(s, d, np.full((len(s), 1), 77, np.uint32))
    g.insert_edges(*_pairs(rng, 300000))
    g.delete_edges(s[::2], d[::2])
    g.close()


@pytest.mark.parametrize("B", [4, 16, 64])
def test_second_graph_on_kept_buffers(B):
    gv = need_gpu()
    say(f"kept buffers, block {B}")
    gv.gv_release_cached()
    _used_graph(gv)
    kept = gv.gv_release_cached()
    assert kept >= 3 * POOL
    _used_graph(gv)
    rng = np.random.default_rng(B)
    s, d = _pairs(rng, 50000)
    g = gv.Graph(N, s, d, block_slots=B, pool_bytes=_pool_bytes(B), edge_attr_words=1)
    o = O.OracleGraph(N, s, d, block_slots=B)
    # the pool came out of what was kept
    assert gv.gv_release_cached() <= kept - 3 * POOL
    assert_same(g, o, "built")
    found, w = g.get_edge_attrs(s[:1000], d[:1000])
    assert found.cpu().numpy().all() and not w.cpu().numpy().any()
    ids = rng.choice(N, 500, replace=False).astype(np.uint32)
    assert g.delete_vertices(ids) == o.delete_vertices(ids)[1]
    assert_same(g, o, "vertices gone")
    assert g.insert_vertices(ids) == o.insert_vertices(ids)[1]
    a, b = _pairs(rng, 200000)
    assert g.insert_edges(a, b) == o.insert_edges(a, b)[1]
    same_answers(g, o, b, a)
    found, w = g.get_edge_attrs(a, b)
    assert not w.cpu().numpy().any()
    assert g.delete_edges(a[::3], b[::3]) == o.delete_edges(a[::3], b[::3])[1]
    assert_same(g, o, "updated")
    g.close()


def test_allocation_that_fails_leaves_the_library_usable():
    """A pool that no card holds: the kept buffers are given back first, and
    the error stays with its call."""
    gv = need_gpu()
    rng = np.random.default_rng(5)
    s, d = _pairs(rng, 20000)
    g = gv.Graph(N, s, d, block_slots=8)
    o = O.OracleGraph(N, s, d, block_slots=8)
    _used_graph(gv)
    with pytest.raises(gv.GraphVineError) as e:
        gv.Graph(N, s, d, block_slots=16, pool_bytes=1 << 41)
    assert e.value.code == gv.GV_ENOMEM
    assert gv.gv_release_cached() < POOL  # (what the failed graph had taken)
    a, b = _pairs(rng, 30000)
    assert g.insert_edges(a, b) == o.insert_edges(a, b)[1]
    assert g.sync() == 0
    assert_same(g, o, "after the failed allocation")
    g.close()
