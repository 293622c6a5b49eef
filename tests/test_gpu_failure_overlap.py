"""A sort that fails on the side stream, forced from the host, while the
graph's stream still applies the batches before it.

With gv_debug_spin_limit(0) every look-back wait of a batch sort gives up at
once; a sort of one tile has none, so batches of at most 2048 pairs sort all
the same (small_sort_max 0 sends them through the passes).  The failure belongs
to its own batch: every batch queued before it is applied whole, it and what
follows changes nothing, and the next synchronising call reports it.  Every
kernel exits normally."""
import numpy as np
import pytest
import torch

from gpu_helpers import assert_same, need_gpu, say
from oracle import pyoracle as O

pytestmark = pytest.mark.gpu

N, B = 1 << 13, 8


def _pairs(rng, size):
    return tuple(rng.integers(0, N, size).astype(np.uint32) for _ in range(2))


def _graphs(gv, rng):
    s, d = _pairs(rng, 60000)
    g = gv.Graph(N, s, d, block_slots=B)
    o = O.OracleGraph(N, s, d, block_slots=B)
    return g, o, (s, d)


def _apply(gv, o, ops):
    for kind, a, b in ops:
        if kind == gv.OP_INSERT_VERTICES:
            o.insert_vertices(a)
        else:
            (o.insert_edges if kind == gv.OP_INSERT_EDGES else o.delete_edges)(a, b)


def _reported(gv, g):
    assert g.sync() == gv.GV_EDEVICE
    with pytest.raises(gv.GraphVineError) as e:
        g.insert_edges([1], [2])
    assert e.value.code == gv.GV_EDEVICE


@pytest.mark.parametrize("form", ["eager", "plan"])
@pytest.mark.parametrize("last", ["insert", "delete"])
@pytest.mark.parametrize("good", [1, 2, 30])
def test_batches_before_a_failed_sort_are_whole(good, last, form):
    gv = need_gpu()
    say(f"failed sort behind {good} batches, {last}, {form}")
    rng = np.random.default_rng(good)
    g, o, have = _graphs(gv, rng)
    gv.gv_set_tuning(g.h, overlap=1, small_sort_max=0)
    ops = []
    for k in range(good):
        pick = rng.integers(0, len(have[0]), 2048)
        ops.append((gv.OP_INSERT_EDGES, *_pairs(rng, 2048)) if k % 2 == 0 else
                   (gv.OP_DELETE_EDGES, have[0][pick], have[1][pick]))
    kind = gv.OP_INSERT_EDGES if last == "insert" else gv.OP_DELETE_EDGES
    bad = [(kind, *_pairs(rng, 60000)), (gv.OP_INSERT_EDGES, *_pairs(rng, 2048))]
    gv.gv_debug_spin_limit(g.h, 0)
    if form == "plan":
        keep = gv.Plan(g.h, ops + bad, g.device)
        keep.launch()
    else:
        keep = gv.gv_apply_ops(g.h, ops + bad, g.device)
    torch.cuda.synchronize()
    _apply(gv, o, ops)
    assert_same(g, o, "as the batches before the failed one left it")
    _reported(gv, g)
    del keep
    g.close()


@pytest.mark.parametrize("runs", [1, 2, 12])
def test_lists_before_a_failed_sort_are_whole(runs):
    """The same for coalesced runs, whose mixed lists sort by rank up to 16384
    entries and by the passes beyond."""
    gv = need_gpu()
    say(f"failed sort behind {runs} lists")
    rng = np.random.default_rng(runs)
    g, o, have = _graphs(gv, rng)
    gv.gv_set_tuning(g.h, overlap=1, coalesce=1)
    ops = []
    for k in range(runs):
        pick = rng.integers(0, len(have[0]), 4000)
        ops += [(gv.OP_INSERT_EDGES, *_pairs(rng, 4000)),
                (gv.OP_DELETE_EDGES, have[0][pick], have[1][pick]),
                (gv.OP_INSERT_VERTICES, np.arange(9, dtype=np.uint32), None)]
    bad = [(gv.OP_INSERT_EDGES, *_pairs(rng, 30000)), (gv.OP_DELETE_EDGES, *_pairs(rng, 30000))]
    gv.gv_debug_spin_limit(g.h, 0)
    keep = gv.gv_apply_ops(g.h, [(*op, gv.OP_FIT_TABLE if op[2] is None else 0)
                                 for op in ops + bad], g.device)
    torch.cuda.synchronize()
    _apply(gv, o, ops)
    assert_same(g, o, "as the lists before the failed one left it")
    _reported(gv, g)
    del keep
    g.close()


@pytest.mark.parametrize("stats", [False, True])
def test_failed_list_changes_nothing(stats):
    gv = need_gpu()
    say(f"failed mixed list, statistics {stats}")
    rng = np.random.default_rng(3)
    g, o, _ = _graphs(gv, rng)
    gv.gv_debug_spin_limit(g.h, 0)
    s, d = _pairs(rng, 50000)
    op = rng.integers(0, 2, 50000).astype(np.uint8)
    keep = (g.apply_edge_ops_stats(op, s, d, [20000, 50000]) if stats
            else g.apply_edge_ops(op, s, d))
    torch.cuda.synchronize()
    assert_same(g, o, "unchanged")
    _reported(gv, g)
    del keep
    g.close()
