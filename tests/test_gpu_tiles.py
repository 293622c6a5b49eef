"""Edge batches at the edges of their tiles: sizes on both sides of the rank
sort's limit, of the tile sizes and of the workgroup sizes; segments that start
and end anywhere in a tile, and that run through many tiles (all pairs of a
batch on one to three sources).  Every batch is compared with the oracle:
statistics, dump, block accounting, audit, answers."""
import numpy as np
import pytest
import torch

from gpu_helpers import assert_same, need_gpu, same_answers, say
from oracle import pyoracle as O

pytestmark = pytest.mark.gpu


def _pairs(rng, n, size, sources, repeat):
    """`size` pairs on `sources` sources (all vertices when 0), a share of
    them repeated, some with ids past the table."""
    s = (rng.integers(0, n, size) if not sources
         else rng.choice(rng.choice(n, sources, replace=False), size))
    d = rng.integers(0, n, size)
    again = rng.integers(0, size, int(repeat * size))
    s[: len(again)], d[: len(again)] = s[again], d[again]
    bad = rng.integers(0, size, size // 50)
    d[bad] += n
    p = rng.permutation(size)
    return s[p].astype(np.uint32), d[p].astype(np.uint32)


# 64 positions per tile up to 2^15 pairs, then 128 and so on up to 4096 past
# 2^20; 256 threads per workgroup up to 1024 positions, 1024 beyond; rank sort
# up to 16384
SIZES = [1, 2, 63, 64, 65, 255, 256, 257, 1023, 4097, 16383, 16384, 16385, 32768, 32769, 131073,
         524288, 524289]


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("sources", [0, 1, 3])
def test_batches_at_tile_edges(size, sources):
    gv = need_gpu()
    say(f"tiles: {size} pairs on {sources or 'all'} sources")
    n, B = 1 << 13, 8
    rng = np.random.default_rng(size * 7 + sources)
    s0, d0 = (rng.integers(0, n, 40000).astype(np.uint32) for _ in range(2))
    g = gv.Graph(n, s0, d0, block_slots=B)
    o = O.OracleGraph(n, s0, d0, block_slots=B)
    ins = _pairs(rng, n, size, sources, 0.2)
    assert g.insert_edges(*ins) == o.insert_edges(*ins)[1]
    assert_same(g, o, "insert")
    same_answers(g, o, *_pairs(rng, n, size, sources, 0.2), "any")
    same_answers(g, o, *ins, "inserted")
    half = rng.permutation(size)[: (size + 1) // 2]
    dele = tuple(a[half] for a in ins)
    assert g.delete_edges(*dele) == o.delete_edges(*dele)[1]
    assert_same(g, o, "delete")
    assert g.insert_edges(*ins) == o.insert_edges(*ins)[1]
    assert g.delete_edges(*ins) == o.delete_edges(*ins)[1]
    assert_same(g, o, "insert and delete again")
    g.close()


@pytest.mark.parametrize("n", [1, 2, 1 << 20, 1 << 25])
def test_small_batches_on_small_and_large_tables(n):
    """The rank sort's keys take 2 log2(n) bits, from none to 50."""
    gv = need_gpu()
    say(f"rank sort on {n} vertices")
    rng = np.random.default_rng(n % 1000)
    hub = rng.integers(0, n, 5)
    g = gv.Graph(n, [], [], block_slots=4)
    o = O.OracleGraph(n, [], [], block_slots=4)
    for size in (1, 300, 5000):
        s = np.where(rng.random(size) < 0.5, rng.choice(hub, size), rng.integers(0, n, size))
        d = rng.integers(0, n + 1, size)
        s, d = s.astype(np.uint32), d.astype(np.uint32)
        assert g.insert_edges(s, d) == o.insert_edges(s, d)[1]
        same_answers(g, o, np.concatenate([s, d]), np.concatenate([d, s]))
        assert g.delete_edges(s[::3], d[::3]) == o.delete_edges(s[::3], d[::3])[1]
        assert (g.memory_used()["blocks_in_use"], g.audit()) == (o.blocks_in_use, 0)
    if n <= 1 << 20:
        assert_same(g, o)
    g.close()


@pytest.mark.parametrize("small", [0, 1, 700, 4096])
def test_sort_by_tuning(small):
    """small_sort_max picks the sort: the radix passes from 0, the rank sort
    up to the limit given."""
    gv = need_gpu()
    n = 3000
    rng = np.random.default_rng(small)
    g = gv.Graph(n, [], [], block_slots=8)
    o = O.OracleGraph(n, [], [], block_slots=8)
    gv.gv_set_tuning(g.h, small_sort_max=small)
    for size in (1, 2, 700, 701, 9000):
        s, d = _pairs(rng, n, size, 0, 0.1) if size > 60 else (
            np.arange(size, dtype=np.uint32), np.arange(size, dtype=np.uint32))
        assert g.insert_edges(s, d) == o.insert_edges(s, d)[1]
        assert g.delete_edges(s[: size // 2], d[: size // 2]) == o.delete_edges(
            s[: size // 2], d[: size // 2])[1]
    assert_same(g, o)
    g.close()
