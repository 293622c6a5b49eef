"""A statistics call behind work that runs far longer than the call polls for:
the poll gives up and the call synchronises."""
import time

import numpy as np
import pytest
import torch

from gpu_helpers import assert_same, need_gpu, say
from oracle import pyoracle as O

pytestmark = pytest.mark.gpu


def _cycles(ms):
    """Sleep cycles of about `ms` milliseconds on this device."""
    torch.cuda._sleep(1000)
    torch.cuda.synchronize()
    t = time.perf_counter()
    torch.cuda._sleep(100000)
    torch.cuda.synchronize()
    return int(100000 * ms * 1e-3 / (time.perf_counter() - t))


def test_statistics_behind_a_long_kernel():
    gv = need_gpu()
    n = 1 << 12
    rng = np.random.default_rng(7)
    s, d = (rng.integers(0, n, 5000).astype(np.uint32) for _ in range(2))
    g = gv.Graph(n, [], [], block_slots=8)
    o = O.OracleGraph(n, [], [], block_slots=8)
    ts, td, ids = (gv.as_device_u32(x, g.device) for x in (s, d, s[:100]))
    cycles = _cycles(20)
    for call, args, want in (("insert_edges", (ts, td), lambda: o.insert_edges(s, d)),
                             ("delete_vertices", (ids,), lambda: o.delete_vertices(s[:100])),
                             ("insert_vertices", (ids,), lambda: o.insert_vertices(s[:100])),
                             ("delete_edges", (td, ts), lambda: o.delete_edges(d, s))):
        torch.cuda.synchronize()
        torch.cuda._sleep(cycles)
        t = time.perf_counter()
        got = getattr(g, call)(*args)
        waited = time.perf_counter() - t
        say(f"{call} behind a kernel: {waited * 1e3:.1f} ms")
        assert got == want()[1], call
        assert waited > 5e-3, call  # the poll ends after 1 ms
    assert_same(g, o)
    g.close()
