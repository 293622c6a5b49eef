"""The probe at the edges of its work items: adjacencies around 128 slots (two
per lane), around a step of 256 and around several items; batch segments
around the 127 entries that are staged whole, and with every second, fourth
and sixteenth entry staged.  Insert, query, delete and delete again, compared
with the oracle."""
import numpy as np
import pytest

from gpu_helpers import assert_same, need_gpu, same_answers, say
from oracle import pyoracle as O

pytestmark = pytest.mark.gpu

DEGS = [1, 8, 9, 33, 127, 128, 129, 131, 255, 256, 257, 385, 511, 513, 1100]
LENS = [1, 8, 9, 63, 126, 127, 128, 129, 254, 255, 509, 2033]


@pytest.mark.parametrize("B", [1, 2, 4, 64])
@pytest.mark.parametrize("chunk", [64, 256, 1024])
def test_items_and_segments(B, chunk):
    gv = need_gpu()
    say(f"probe items: block {B}, chunk {chunk}")
    n = 4096
    rng = np.random.default_rng(B * 10 + chunk)
    src = np.arange(len(DEGS))
    dst = [rng.choice(n, d, replace=False) for d in DEGS]
    s0 = np.repeat(src, DEGS).astype(np.uint32)
    d0 = np.concatenate(dst).astype(np.uint32)
    for k, ln in enumerate(LENS):
        g = gv.Graph(n, s0, d0, block_slots=B)
        o = O.OracleGraph(n, s0, d0, block_slots=B)
        gv.gv_set_tuning(g.h, item_chunk=chunk)
        s, d = [], []
        for v, have in zip(src, dst):
            # half of the segment from the adjacency (its first and last slots
            # among them), the rest anything; every seventh entry repeated
            old = np.concatenate([have[:1], have[-1:], rng.choice(have, ln)])[: (ln + 1) // 2]
            e = np.concatenate([old, rng.integers(0, n, ln)])[:ln]
            e[6::7] = e[5::7][: len(e[6::7])]
            s.append(np.full(ln, v))
            d.append(e)
        p = rng.permutation(ln * len(src))
        s = np.concatenate(s)[p].astype(np.uint32)
        d = np.concatenate(d)[p].astype(np.uint32)
        same_answers(g, o, s, d, f"segments of {ln}")
        first, second = [("insert_edges", "delete_edges"), ("delete_edges", "insert_edges")][k % 2]
        for call in (first, first, second):
            assert getattr(g, call)(s, d) == getattr(o, call)(s, d)[1], (call, ln)
            assert_same(g, o, f"{call}, segments of {ln}")
        g.close()
