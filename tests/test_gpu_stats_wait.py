"""Statistics waits: with an idle stream, and behind a queue of batches that
runs longer than the wait polls for."""
import numpy as np
import pytest
import torch

from gpu_helpers import assert_same, need_gpu, say
from oracle import pyoracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("queued", [0, 1, 40])
def test_stats_behind_a_queue(queued):
    gv = need_gpu()
    say(f"statistics behind {queued} queued batches")
    n, size = 1 << 14, 200000
    rng = np.random.default_rng(queued)
    pairs = [tuple(rng.integers(0, n, size).astype(np.uint32) for _ in range(2)) for _ in range(4)]
    dev = [tuple(torch.from_numpy(a.view(np.int32)).cuda() for a in p) for p in pairs]
    g = gv.Graph(n, [], [], block_slots=16)
    o = O.OracleGraph(n, [], [], block_slots=16)
    for k in range(queued):
        (g.insert_edges if k % 2 == 0 else g.delete_edges)(*dev[k % 4], stats=False)
        (o.insert_edges if k % 2 == 0 else o.delete_edges)(*pairs[k % 4])
    last = tuple(a[: size // 2] for a in pairs[1])
    assert g.insert_edges(*last) == o.insert_edges(*last)[1]
    ids = rng.integers(0, n, 300).astype(np.uint32)
    assert g.delete_vertices(ids) == o.delete_vertices(ids)[1]
    assert g.insert_vertices(ids) == o.insert_vertices(ids)[1]
    assert_same(g, o)
    g.close()
