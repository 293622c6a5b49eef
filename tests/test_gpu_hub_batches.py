"""Batches that lie on one vertex or a few, in tiles of every size: their plan
counts a segment of hundreds of tiles.  Results against set algebra, and the
plan's time against that of a batch spread over the table."""
import numpy as np
import pytest
import torch

from gpu_helpers import EdgeSet, gpu_dump, mix64_sum, need_gpu, say

pytestmark = pytest.mark.gpu

N = 1 << 21


def _star(rng, size, hubs):
    """`size` distinct pairs on `hubs` vertices, the segments about equal."""
    src = np.sort(rng.choice(N, hubs, replace=False))
    s = src[np.arange(size) % hubs]
    return s.astype(np.uint32), rng.permutation(N)[:size].astype(np.uint32)


def _same(g, e, label):
    _, dst, ck, m = gpu_dump(g)
    assert (ck, m) == (mix64_sum(e.E), len(e.E)), label
    np.testing.assert_array_equal(dst, (e.E & np.uint64(0xffffffff)).astype(np.uint32), label)
    assert g.audit() == 0, label


# 64 positions per tile up to 2^15 pairs, 4096 past 2^21; from 2^20 on 1024
# threads a workgroup
@pytest.mark.parametrize("size,hubs", [(20000, 1), (100000, 1), (100003, 2), (300000, 1),
                                       (1060001, 1), (1060001, 3), (2097152, 1), (2097151, 2)])
def test_results(size, hubs):
    gv = need_gpu()
    say(f"hub batch: {size} pairs on {hubs}")
    rng = np.random.default_rng(size + hubs)
    s, d = _star(rng, size, hubs)
    half = rng.permutation(size)[: size // 2]
    g = gv.Graph(N, s[half], d[half], block_slots=16, pool_bytes=1 << 28)
    e = EdgeSet(N, s[half], d[half])
    # every other pair is there already, some come twice
    bs, bd = np.concatenate([s, s[:999]]), np.concatenate([d, d[:999]])
    assert g.insert_edges(bs, bd) == (e.insert(bs, bd), 0, 999)
    _same(g, e, "insert")
    third = rng.permutation(size)[: size // 3]
    g.delete_edges(s[third], d[third])
    e.delete(s[third], d[third])
    _same(g, e, "delete")
    assert g.delete_edges(bs, bd) == (e.delete(bs, bd), 0, 999)
    _same(g, e, "all deleted")
    g.close()


@pytest.mark.parametrize("size", [100000, 1000000])
def test_plan_time_does_not_follow_one_segment(size):
    """The tiles of a segment are counted beside each other: the plan of a
    batch on one vertex takes no more than four times that of a spread one
    (counted by the workgroup of the segment's head it took 5 and 15 times)."""
    gv = need_gpu()
    rng = np.random.default_rng(size)
    hub = [torch.from_numpy(a.view(np.int32)).cuda() for a in _star(rng, size, 1)]
    wide = [torch.from_numpy(rng.integers(0, N, size).astype(np.int32)).cuda() for _ in range(2)]
    us = {}
    for name, (s, d) in (("hub", hub), ("wide", wide)):
        g = gv.Graph(N, s, d, block_slots=16, pool_bytes=1 << 28)
        for _ in range(3):
            g.insert_edges(s, d, stats=False)
        gv.gv_profile_enable(g.h)
        gv.gv_profile_reset(g.h)
        for _ in range(10):
            g.insert_edges(s, d, stats=False)
        n, ms = gv.gv_kernel_times(g.h, "plan_insert")
        us[name] = ms / n * 1e3
        g.close()
    say(f"plan of {size} pairs: {us}")
    assert us["hub"] < 4 * us["wide"], us


@pytest.mark.parametrize("size", [17, 63, 64, 65, 255, 256, 257, 513, 5000, 100003])
def test_few_pairs_many_times(size):
    """A long segment with few hits, in rows of 64 and rounds of 256: one pair,
    and five of which the last slots of the adjacency are two."""
    gv = need_gpu()
    say(f"few pairs, {size} entries")
    rng = np.random.default_rng(size)
    deg = 40
    d0 = rng.choice(N, deg, replace=False)
    s0 = np.full(deg, 99)
    for picks in (d0[:1], np.concatenate([d0[:3], d0[-2:]])):
        g = gv.Graph(N, s0, d0, block_slots=8, pool_bytes=1 << 26)
        e = EdgeSet(N, s0, d0)
        d = np.sort(rng.choice(picks, size))
        s = np.full(size, 99)
        hits = len(np.unique(d))
        assert g.delete_edges(s, d) == (e.delete(s, d), 0, size - hits)
        _same(g, e, "deleted")
        assert g.insert_edges(s, d) == (e.insert(s, d), 0, size - hits)
        _same(g, e, "inserted")
        g.close()
