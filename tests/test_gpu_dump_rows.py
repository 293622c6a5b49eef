"""Canonical dumps and bulk builds at the edges of the row classes: a row is
ordered by 16 lanes, a wave in registers, a workgroup's bitmap windows, a
workgroup in LDS or the device-wide sort, by its degree and the table's size.  Whole numbers: compared exactly with
numpy's sort of the same pairs."""
import numpy as np
import pytest
import torch

from gpu_helpers import gpu_dump, mix64_sum, keys_of, need_gpu, say

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 15, 16, 17, 63, 64, 65, 127, 128, 129, 1023, 1024, 1025, 2049, 16383, 16384, 16385,
         40000]


def _rows(degrees, n, seed, repeat):
    """One vertex per degree (spread over the table), distinct destinations in
    random order, a share of the pairs handed in twice."""
    rng = np.random.default_rng(seed)
    ids = np.sort(rng.choice(n, len(degrees), replace=False))
    src = np.repeat(ids, degrees)
    dst = np.concatenate([rng.choice(n, d, replace=False) for d in degrees])
    again = rng.choice(len(src), int(repeat * len(src)), replace=False)
    s, d = np.concatenate([src, src[again]]), np.concatenate([dst, dst[again]])
    p = rng.permutation(len(s))
    return s[p].astype(np.uint32), d[p].astype(np.uint32)


@pytest.mark.parametrize("log_n,block,degrees", [
    (17, 1, EDGES[:14]), (17, 8, EDGES), (16, 16, [d for d in EDGES for _ in range(3)]),
    (17, 64, EDGES[::-1]), (12, 16, [0, 3, 4096]), (17, 16, [70000, 1, 50000]),
    (17, 1024, [64, 65, 20000]), (20, 16, [1025, 90000]), (21, 16, [1024, 1025, 30000, 7]),
    (22, 8, [1025, 100000, 64, 65]), (23, 16, EDGES[8:]), (23, 16, [1025, 16385])])
def test_dump_orders_rows_of_every_class(log_n, block, degrees):
    gv = need_gpu()
    say(f"dump rows: 2^{log_n} vertices, block {block}, degrees {degrees}")
    n = 1 << log_n
    s, d = _rows(degrees, n, 7 + block, 0.1)
    want = np.unique(keys_of(s, d))
    offs = np.zeros(n + 1, np.uint64)
    np.cumsum(np.bincount((want >> np.uint64(32)).astype(np.int64), minlength=n), out=offs[1:])
    g = gv.Graph(n, s, d, block_slots=block)

    def same(label):
        go, gd, ck, e = gpu_dump(g)
        np.testing.assert_array_equal(go, offs, err_msg=label)
        np.testing.assert_array_equal(gd, (want & np.uint64(0xffffffff)).astype(np.uint32),
                                      err_msg=label)
        assert (ck, e) == (mix64_sum(want), len(want)), label
        assert g.dump(checksum_only=True)[2:] == (ck, e), label
        assert g.audit() == 0, label

    same("built")
    # take every other stored pair away and hand it back: rows out of order,
    # freed blocks with stale owners
    half = want[::2]
    hs, hd = (half >> np.uint64(32)).astype(np.uint32), half.astype(np.uint32)
    g.delete_edges(hs, hd)
    _, _, ck, e = g.dump(checksum_only=True)
    assert (ck, e) == (mix64_sum(want[1::2]), len(want) - len(half)), "half"
    p = np.random.default_rng(1).permutation(len(hs))
    g.insert_edges(hs[p], hd[p])
    same("given back")
    g.close()


@pytest.mark.parametrize("m", [0, 1, 2, 4095, 4097])
def test_build_of_few_pairs(m):
    gv = need_gpu()
    say(f"build of {m} pairs")
    rng = np.random.default_rng(m)
    for n in (1, 2, 1000):
        s, d = (rng.integers(0, n, m).astype(np.uint32) for _ in range(2))
        g = gv.Graph(n, s, d, block_slots=4)
        want = np.unique(keys_of(s, d))
        offs, dst, ck, e = gpu_dump(g)
        np.testing.assert_array_equal(dst, (want & np.uint64(0xffffffff)).astype(np.uint32))
        assert (ck, e) == (mix64_sum(want), len(want))
        assert g.audit() == 0
        g.close()
    with pytest.raises(gv.GraphVineError) as x:
        gv.Graph(5, np.array([1] * max(m, 1)), np.array([5] * max(m, 1)))
    assert x.value.code == gv.GV_ERANGE
