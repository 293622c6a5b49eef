"""The workloads the library's speed is judged on: what a program that keeps a
dynamic graph on the GPU has it do, over the range of sizes it does it with.

Every case is a graph (R-MAT of 2^scale vertices, or a road-like lattice) and
one kind of call on it:

  updates   a stream of edge insert and delete batches, with or without
            statistics per batch
  query     a batch of pair queries
  attrs     attribute words written to and read from stored edges
  vertices  vertices deleted, inserted again and given their edges back
  mixed     lists of inserts and deletes cut into requests, with statistics
            per request (a tick of a server)
  plan      a recorded sequence of batches of uneven sizes
  build     a graph made from a COO list and read back as canonical CSR

Inputs are drawn on the GPU from seeded counter-based streams.  The update
workloads are cyclic: what one pass inserts and deletes, the pass (or the one
after it) takes back, so that a pass does the same work however often it runs.
"""
import math
import random

import torch

from paper_2306_08252_amd import graphvine as gv
from paper_2306_08252_amd import inputs as I
from paper_2306_08252_amd import inputs_torch as T

DEV = "cuda:0"
SAMPLE = 20000  # pairs asked after a recorded sequence, which returns nothing itself
# the settings the autotuner stored for streams of large batches
STREAM = {"overlap": 1, "item_chunk": 512}


def listed():
    return [
        # the smallest updates: a client that sends a thousand pairs and waits
        # for the counts
        dict(name="updates_1e3_stats", kind="updates", graph="rmat", scale=20, edges=1 << 24,
             block=16, n=1000, steps=4, stats=True, tuned=False),
        # small batches queued one after the other, default settings
        dict(name="updates_1e4", kind="updates", graph="rmat", scale=20, edges=1 << 24, block=32,
             n=10007, steps=4, stats=False, tuned=False),
        # road-like graph (low degrees, blocks of 8), ragged batches, counts read
        dict(name="updates_lattice_1e5", kind="updates", graph="lattice", scale=22, edges=0,
             block=8, n=131101, steps=2, stats=True, tuned=False),
        # the headline: streams of 10^6-pair batches on the power-law graph
        dict(name="updates_1e6", kind="updates", graph="rmat", scale=20, edges=1 << 24, block=16,
             n=10**6, steps=4, stats=False, tuned=True),
        # the largest batches, on a larger graph
        dict(name="updates_1e7", kind="updates", graph="rmat", scale=22, edges=1 << 26, block=16,
             n=10**7, steps=2, stats=False, tuned=False),
        # a lookup of a couple of thousand pairs, and a large one
        dict(name="query_2e3", kind="query", graph="rmat", scale=20, edges=1 << 24, block=16,
             n=2000),
        dict(name="query_1e6", kind="query", graph="rmat", scale=20, edges=1 << 24, block=16,
             n=10**6),
        # weighted graph: two words per edge written and read
        dict(name="attrs_1e5", kind="attrs", graph="rmat", scale=20, edges=1 << 22, block=16,
             n=100003, words=2),
        # a batch of vertices leaves and comes back
        dict(name="vertices_1e4", kind="vertices", graph="rmat", scale=20, edges=1 << 24,
             block=16, n=10**4),
        # a busy server's tick: some tens of clients' requests in one list
        dict(name="mixed_2e5", kind="mixed", graph="rmat", scale=20, edges=1 << 24, block=16,
             n=200003, requests=40),
        # uneven batches, recorded once and launched as one
        dict(name="plan_24", kind="plan", graph="rmat", scale=20, edges=1 << 24, block=16,
             batches=24, lo=100, hi=10**6),
        # load a graph and hand it on as CSR
        dict(name="build_csr", kind="build", graph="rmat", scale=20, edges=1 << 24, block=16),
    ]


def _log(rng, lo, hi):
    return int(round(lo * math.exp(rng.random() * math.log(hi / lo))))


def draw(rng: random.Random):
    kind = rng.choice(["updates", "updates", "updates", "query", "attrs", "vertices", "mixed",
                       "plan", "build"])
    lattice = kind in ("updates", "query") and rng.random() < 0.3
    scale = rng.choice([18, 20, 22]) if lattice else rng.randint(16, 21)
    c = dict(kind=kind, graph="lattice" if lattice else "rmat", scale=scale,
             edges=0 if lattice else (1 << scale) * rng.choice([4, 8, 16]),
             block=rng.choice([8, 16, 32, 64]))
    if kind == "updates":
        c.update(n=_log(rng, 500, 2 * 10**6), steps=rng.choice([2, 4]),
                 stats=rng.random() < 0.4, tuned=rng.random() < 0.4)
    elif kind == "query":
        c.update(n=_log(rng, 500, 2 * 10**6))
    elif kind == "attrs":
        c.update(n=_log(rng, 1000, 10**6), words=rng.randint(1, 3))
    elif kind == "vertices":
        c.update(n=_log(rng, 100, 2 * 10**4))
    elif kind == "mixed":
        c.update(n=_log(rng, 1000, 10**6), requests=rng.randint(1, 64))
    elif kind == "plan":
        c.update(batches=rng.randint(8, 24), lo=100, hi=_log(rng, 10**4, 10**6))
    return c


# ------------------------------------------------------------------ inputs
def _num_vertices(case):
    return 1 << case["scale"]


def _seed(case, seed, *what):
    return I.stream_seed("perf", case["kind"], case["graph"], case["scale"], seed, *what)


def _graph_pairs(case, seed):
    """The initial COO list.  R-MAT lists hold some repeated pairs, as a list
    that was never cleaned does; a build takes distinct pairs, so that every
    seed's graph has the same number of edges."""
    if case["kind"] == "build":
        return T.rmat_graph(_seed(case, seed, "graph"), case["scale"], case["edges"], device=DEV)
    if case["graph"] == "rmat":
        return T.rmat_pairs(_seed(case, seed, "graph"), case["edges"], case["scale"], device=DEV)
    # 4-neighbour lattice, a tenth of its edges taken out, one in a hundred
    # added between any two vertices; stored in both directions
    nv = _num_vertices(case)
    side = 1 << (case["scale"] // 2)
    v = torch.arange(nv, dtype=torch.int64, device=DEV)
    right, down = v[v % side != side - 1], v[v < nv - side]
    s = torch.cat([right, down])
    d = torch.cat([right + 1, down + side])
    keep = T.splitmix64(_seed(case, seed, "drop"), s.numel(), device=DEV) % 10 != 0
    s, d = s[keep].to(torch.int32), d[keep].to(torch.int32)
    ls, ld = T.uniform_pairs(_seed(case, seed, "long"), s.numel() // 100, nv, device=DEV)
    s, d = torch.cat([s, ls]), torch.cat([d, ld])
    return torch.cat([s, d]), torch.cat([d, s])


def _new_pairs(case, seed, n, *what):
    """Pairs that an insert batch brings: R-MAT pairs, or uniform pairs."""
    if case["graph"] == "rmat":
        return T.rmat_pairs(_seed(case, seed, "new", *what), n, case["scale"], device=DEV)
    return T.uniform_pairs(_seed(case, seed, "new", *what), n, _num_vertices(case), device=DEV)


def _batches(case, seed, sizes, src, dst):
    """Insert and delete batches of about the given sizes.  Step j inserts new
    pairs R_j and the old edges E_(j-1) that the step before deleted, and
    deletes old edges E_j, the new pairs R_(j-1), and a fifth of uniform
    pairs, nearly all of them absent; the last step is before the first."""
    new, old = [], []
    for j, n in enumerate(sizes):
        new.append(_new_pairs(case, seed, n // 2, j))
        old.append(T.pick(_seed(case, seed, "old", j), max(1, 2 * n // 5), src, dst))
    out = []
    for j, n in enumerate(sizes):
        ins = [torch.cat(p) for p in zip(new[j], old[j - 1])]
        absent = T.uniform_pairs(_seed(case, seed, "absent", j), n // 5, _num_vertices(case),
                                 device=DEV)
        dele = [torch.cat(p) for p in zip(old[j], new[j - 1], absent)]
        out.append((T.shuffle_pairs(_seed(case, seed, "mix-ins", j), *ins),
                    T.shuffle_pairs(_seed(case, seed, "mix-del", j), *dele)))
    return out


def _queries(case, seed, n, src, dst):
    """Half of the pairs stored, half uniform, shuffled."""
    es, ed = T.pick(_seed(case, seed, "query-old"), n // 2, src, dst)
    us, ud = T.uniform_pairs(_seed(case, seed, "query-any"), n - n // 2, _num_vertices(case),
                             device=DEV)
    return T.shuffle_pairs(_seed(case, seed, "query-mix"), torch.cat([es, us]),
                           torch.cat([ed, ud]))


def _words(case, seed, n):
    r = T.splitmix64(_seed(case, seed, "words"), n * case["words"], device=DEV)
    return r.to(torch.int32).reshape(n, case["words"])


def _request_ends(case, seed):
    """Ends of `requests` requests of log-uniform sizes that add up to n."""
    rng = random.Random(_seed(case, seed, "requests"))
    r, n = case["requests"], case["n"]
    w = [math.exp(rng.random() * math.log(1000)) for _ in range(r)]
    total, run, ends = sum(w), 0.0, []
    for x in w:
        run += x
        ends.append(min(n, int(round(n * run / total))))
    ends[-1] = n
    return torch.tensor(ends, dtype=torch.int64, device=DEV)


# ------------------------------------------------------------------ state
def prepare(case, seed):
    src, dst = _graph_pairs(case, seed)
    st = dict(case=case, nv=_num_vertices(case))
    if case["kind"] == "build":
        st.update(src=src, dst=dst)
        return st
    g = gv.Graph(st["nv"], src, dst, block_slots=case["block"], device=DEV,
                 edge_attr_words=case.get("words", 0))
    st["g"] = g
    kind = case["kind"]
    if kind == "updates":
        if case["tuned"]:
            gv.gv_set_tuning(g.h, **STREAM)
        st["batches"] = _batches(case, seed, [case["n"]] * case["steps"], src, dst)
        st["ask"] = _queries(case, seed, max(1, case["n"] // 8), src, dst)
    elif kind == "query":
        st["ask"] = _queries(case, seed, case["n"], src, dst)
    elif kind == "attrs":
        st["ask"] = _queries(case, seed, case["n"], src, dst)
        st["words"] = _words(case, seed, case["n"])
    elif kind == "vertices":
        order = T.permutation(_seed(case, seed, "ids"), st["nv"], DEV)
        ids = order[: case["n"]]
        gone = torch.zeros(st["nv"], dtype=torch.bool, device=DEV)
        gone[ids] = True
        back = gone[src.long()] | gone[dst.long()]
        st.update(ids=ids.to(torch.int32), src=src[back].contiguous(),
                  dst=dst[back].contiguous())
    elif kind == "mixed":
        (ins, dele), = _batches(case, seed, [case["n"]], src, dst)
        ni = case["n"] // 2
        s = torch.cat([ins[0][:ni], dele[0][: case["n"] - ni]])
        d = torch.cat([ins[1][:ni], dele[1][: case["n"] - ni]])
        op = torch.zeros(s.numel(), dtype=torch.uint8, device=DEV)
        op[ni:] = 1
        p = T.permutation(_seed(case, seed, "order"), s.numel(), DEV)
        st.update(op=op[p].contiguous(), src=s[p].contiguous(), dst=d[p].contiguous(),
                  ends=_request_ends(dict(case, n=s.numel()), seed))
        st["undo"] = 1 - st["op"]  # the tick after it takes the changes back
    elif kind == "plan":
        gv.gv_set_tuning(g.h, coalesce=1, max_run_pairs=1 << 22, **STREAM)
        rng = random.Random(_seed(case, seed, "sizes"))
        sizes = [_log(rng, case["lo"], case["hi"]) for _ in range(case["batches"] // 2)]
        ops = []
        for j, (ins, dele) in enumerate(_batches(case, seed, sizes, src, dst)):
            ops.append((gv.OP_INSERT_EDGES, *ins))
            ops.append((gv.OP_DELETE_EDGES, *dele))
            if j % 6 == 5:  # now and then some vertices leave and come back empty
                ids = (T.splitmix64(_seed(case, seed, "leave", j), 1000, device=DEV)
                       & (st["nv"] - 1)).to(torch.int32)
                ops.append((gv.OP_DELETE_VERTICES, ids, None))
                ops.append((gv.OP_INSERT_VERTICES, ids, None))
        st["ask"] = _queries(case, seed, SAMPLE, src, dst)
        g.edge_exists(*st["ask"])  # one eager run sizes the buffers that the recording holds
        gv.gv_apply_ops(g.h, ops, DEV)
        st["plan"] = gv.Plan(g.h, ops, DEV)
    return st


def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "build":
        g = gv.Graph(st["nv"], st["src"], st["dst"], block_slots=case["block"], device=DEV)
        offsets, dst, checksum, edges = g.dump()
        blocks = g.memory_used()["blocks_in_use"]
        g.close()
        return offsets, dst, checksum - (1 << 64) if checksum >> 63 else checksum, edges, blocks
    g = st["g"]
    if kind == "updates":
        counts = []
        for ins, dele in st["batches"]:
            counts.append(g.insert_edges(*ins, stats=case["stats"]))
            counts.append(g.delete_edges(*dele, stats=case["stats"]))
        return counts if case["stats"] else g.edge_exists(*st["ask"])
    if kind == "query":
        return g.edge_exists(*st["ask"])
    if kind == "attrs":
        g.set_edge_attrs(*st["ask"], st["words"], stats=False)
        return g.get_edge_attrs(*st["ask"])
    if kind == "vertices":
        return [g.delete_vertices(st["ids"]), g.insert_vertices(st["ids"]),
                g.insert_edges(st["src"], st["dst"])]
    if kind == "mixed":
        _, first = g.apply_edge_ops_stats(st["op"], st["src"], st["dst"], st["ends"])
        _, back = g.apply_edge_ops_stats(st["undo"], st["src"], st["dst"], st["ends"])
        return first, back
    st["plan"].launch()
    return g.edge_exists(*st["ask"])


# ------------------------------------------------------------------ work
def _touched_slots(case, n):
    """Adjacency entries of the sources that n pairs touch: each has to be
    read once, an adjacency being an unordered set.  Uniform sources: n times
    the mean degree, at most every edge.  R-MAT: a source whose row takes the
    less likely half of the matrix at k of its levels is drawn with
    probability p^k (1 - p)^(scale - k), p = 0.24."""
    nv, scale = _num_vertices(case), case["scale"]
    if case["graph"] == "lattice":
        return int(4 * nv * 0.9 * (1 - math.exp(-n / nv)))
    total = 0.0
    for k in range(scale + 1):
        q = 0.24**k * 0.76**(scale - k)
        total += math.comb(scale, k) * q * (1 - math.exp(-n * q))
    return int(case["edges"] * total)


def _batch_bytes(case, n):
    # the pairs, the touched adjacencies, and a slot written for most pairs
    return 8 * n + 4 * _touched_slots(case, n) + 3 * n


def work(case):
    kind = case["kind"]
    if kind == "updates":
        b = 2 * case["steps"] * _batch_bytes(case, case["n"])
        if not case["stats"]:
            b += 9 * (case["n"] // 8) + 4 * _touched_slots(case, case["n"] // 8)
    elif kind == "query":
        b = 9 * case["n"] + 4 * _touched_slots(case, case["n"])
    elif kind == "attrs":
        n = case["n"]
        b = 2 * (8 * n + 4 * _touched_slots(case, n)) + n + 16 * n * case["words"]
    elif kind == "vertices":
        # every stored destination is looked at once; about the mean degree of
        # edges out of and into each vertex goes and comes back
        moved = 2 * case["n"] * case["edges"] // _num_vertices(case)
        b = 4 * case["edges"] + 8 * case["n"] + 8 * moved
        b += _batch_bytes(case, moved)
    elif kind == "mixed":
        b = 2 * (_batch_bytes(case, case["n"]) + case["n"] + 32 * case["requests"])
    elif kind == "plan":
        # the mean of the sizes drawn log-uniformly between lo and hi
        n = int((case["hi"] - case["lo"]) / math.log(case["hi"] / case["lo"]))
        # runs of edge batches between vertex batches may be applied as one:
        # the touched adjacencies once per run
        steps = case["batches"] // 2
        runs = max(1, (steps + 5) // 6)
        b = runs * _batch_bytes(case, 2 * steps * n // runs)
    else:
        m = case["edges"]
        # the list in, the graph's slots out and in again, CSR out
        b = 8 * m + 4 * m + 4 * m + 4 * m + 8 * (_num_vertices(case) + 1)
    return {"bytes": int(b), "flops": 0}


# ------------------------------------------------------------------ plain answers
def exact(case, seed):
    """Plain torch: the answers of queries and the CSR of a build.  The other
    kinds return counts and answers after many batches: whole numbers, with
    no simpler computation than the batches one by one."""
    kind = case["kind"]
    if kind not in ("query", "build"):
        return None
    src, dst = _graph_pairs(case, seed)
    keys = torch.unique(T.pair_keys(src, dst))
    if kind == "query":
        return torch.isin(T.pair_keys(*_queries(case, seed, case["n"], src, dst)),
                          keys).to(torch.uint8)
    nv = _num_vertices(case)
    deg = torch.bincount(keys >> 32, minlength=nv)
    offsets = torch.zeros(nv + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(deg, 0, out=offsets[1:])
    s, d = keys >> 32, keys & 0xFFFFFFFF
    checksum = int(T.mix64((s << 32) | d).sum())
    blocks = int(((deg + case["block"] - 1) // case["block"]).sum())
    return offsets, d.to(torch.int32), checksum, keys.numel(), blocks
