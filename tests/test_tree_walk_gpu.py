"""The one-launch tree walk, export and eviction and the level-by-level kernels
behind them, at the sizes where one hands over to the other, against the CPU
oracle: deep chains, wide levels, more leaves than are sorted in LDS, many
nodes of one time at one depth, times that differ in any byte."""
import numpy as np
import pytest

import pins
from gpu_util import announce, device

pytestmark = pytest.mark.gpu


class Pair:
    """A forest and the oracle given the same operations; peer `local` keeps times."""

    def __init__(self, P, local):
        import oracle
        from paper_2606_17059_amd import Forest
        self.f, self.o, self.P, self.local = Forest(P), oracle.Oracle(P), P, local
        if local >= 0:
            self.f.set_local_peer(local)
            self.o.set_local(local)

    def merge(self, peer, seqs, t=None):
        import torch
        if t is not None:
            self.f.set_time(t)
            self.o.set_time(t)
        tok, off = pins._csr(seqs)
        peers = np.full(len(seqs), peer, np.int32)
        self.f.merge(*[torch.from_numpy(x).to(device()) for x in (peers, tok, off)])
        self.o.merge(peers, tok, off)

    def export(self, p, what):
        announce(f"export {what}")
        t, o = self.f.export_snapshot(p)
        got = sorted(map(tuple, pins.csr_to_list(t.cpu().numpy(), o.cpu().numpy())))
        assert got == sorted(map(tuple, pins.csr_to_list(*self.o.export(p)))), what
        assert self.f.tree_tokens(p) == self.o.tree_tokens(p), what

    def evict(self, n, what):
        announce(f"evict {n} {what}")
        assert self.f.evict_lru(n) == self.o.evict(n), what
        self.export(self.local, what)

    def close(self):
        self.f.close()
        self.o.close()


def _chain(n):
    """Prefixes of one path, so that every token is a node of its own."""
    path = [(7 * i) % 5 for i in range(n)]
    return [path[:k] for k in range(1, n + 1)]


@pytest.mark.parametrize("what,make", [
    ("empty tree", lambda: []),
    ("one token", lambda: [[3]]),
    ("chain of 300", lambda: _chain(300)),
    ("4096 parents", lambda: [[i, 1] for i in range(4096)] + [[i, 2] for i in range(4096)]),
    ("4097 parents", lambda: [[i, 1] for i in range(4097)] + [[i, 2] for i in range(4097)]),
    ("8192 leaves", lambda: [[9, i, i % 7] for i in range(8192)]),
    ("8193 leaves", lambda: [[9, i, i % 7] for i in range(8193)]),
    ("a level of 131073", lambda: [[i] for i in range(131073)]),
])
@pytest.mark.parametrize("peer", [0, 66])
def test_walk_and_export_sizes(what, make, peer):
    p = Pair(67, -1)
    p.merge(1, [[9, 1, 5, 5], [2, 2]])  # paths the exported peer does not hold
    seqs = make()
    if seqs:
        p.merge(peer, seqs)
    p.export(peer, what)
    p.export(1, what)
    p.close()


def test_export_buffers_too_small():
    """Sizes are reported and nothing is written."""
    import ctypes
    import torch
    from paper_2606_17059_amd import router as R
    p = Pair(2, -1)
    p.merge(1, [[1, 2, 3], [1, 5], [4]])
    t = torch.full((8,), -7, dtype=torch.int32, device=device())
    o = torch.full((8,), -7, dtype=torch.int64, device=device())
    for tcap, ocap in ((5, 4), (6, 3), (0, 0)):
        ns, nt = ctypes.c_int64(0), ctypes.c_int64(0)
        st = R.lib().pr_export_snapshot(p.f.handle, 1, t.data_ptr(), tcap, o.data_ptr(), ocap, ctypes.byref(ns),
                                        ctypes.byref(nt), 0)
        assert (st, ns.value, nt.value) == (R.PR_EINVAL, 3, 6), (tcap, ocap)
    torch.cuda.synchronize()
    assert (t == -7).all() and (o == -7).all()
    # no tokens wanted and none there: the offsets alone
    st = R.lib().pr_export_snapshot(p.f.handle, 0, None, 5, o.data_ptr(), 1, ctypes.byref(ns), ctypes.byref(nt), 0)
    torch.cuda.synchronize()
    assert (st, ns.value, nt.value) == (R.PR_OK, 0, 0) and o.cpu().tolist() == [0] + [-7] * 7
    p.close()


@pytest.mark.parametrize("nodes", [40, 4095, 4096, 4097])
def test_eviction_around_the_node_limit(nodes):
    """Trees of about `nodes` nodes; a few tokens at a time from a time class
    that all of them share, then all of an older one."""
    rng = np.random.default_rng(nodes)
    p = Pair(3, 1)
    p.merge(0, [[i, 5, 5, 1] for i in range(30)])
    p.merge(1, [[i] + rng.integers(0, 4, 1 + i % 3).tolist() for i in range(nodes)], t=5)
    for k, n in enumerate((1, 3, 7)):
        p.evict(n, f"{nodes} nodes, eviction {k}")
    p.merge(1, [[i, 5, 5, 1] for i in range(12)], t=9)
    p.evict(11, f"{nodes} nodes, after newer inserts")
    p.export(0, "the other peer")
    p.close()


@pytest.mark.parametrize("width", [1, 2, 512, 513, 700])
def test_ties_at_the_cut_depth(width):
    """`width` paths of one time and length: the lexicographically smallest lose
    their last tokens first, past the width compared in LDS too."""
    p = Pair(2, 0)
    p.merge(0, [[width - i, 3, i % 11, 4] for i in range(width)], t=1)
    p.merge(1, [[2, 3, 1, 4, 8]])
    for n in (1, max(1, width // 2), width, 5):
        p.evict(n, f"{width} ties, {n} tokens")
    p.close()


def test_times_that_differ_in_any_byte():
    p = Pair(2, 0)
    times = sorted({0, 1, 2, 255, 256, 257, 65536, 70000, 1 << 24, (1 << 32) + 3, (1 << 40) + 1, (1 << 55) + 9,
                    (1 << 62) + 77, (1 << 62) + 78})
    for i, t in enumerate(times):
        p.merge(0, [[1, 2, i, j, 6] for j in range(3)], t=t)
    for k, n in enumerate((4, 1, 20, 9, 2, 30, 10 ** 9)):
        p.evict(n, f"times, eviction {k}")
    p.close()


@pytest.mark.parametrize("records", [8191, 8192, 8193])
@pytest.mark.parametrize("P, local", [(2, 0), (67, 66)])
def test_eviction_around_the_record_limit(records, P, local):
    """Sizes and evictions over the records of a loaded forest (the root and a
    record a sequence), with child blocks of 8, 9, 64 and 65 among them; cuts
    and merges then add records and move others."""
    p = Pair(P, local)
    inner = [[5, k, 6, i] for k, c in enumerate((8, 9, 64, 65)) for i in range(c)]
    seqs = inner + [[100 + i, 1, i % 3, 4] for i in range(records - 2 - 4 - len(inner))]
    for q in (p.f, p.o):
        q.set_time(3)
        q.load_snapshot(local, *pins._csr(seqs)) if q is p.f else q.load(local, *pins._csr(seqs))
    p.export(local, "loaded")
    assert p.f.info()["num_nodes"] == records
    for k, n in enumerate((5, 3000, 40)):
        p.evict(n, f"{records} records, eviction {k}")
    p.merge(local, inner[:70] + [[5, 1, 9], [7] * 9], t=8)
    p.merge(1 - local if P == 2 else 1, [[5, 1, 6, 2, 2], [7, 7]])
    p.evict(len(seqs), "after moves")
    p.export(1, "another peer")
    p.close()


def test_eviction_from_a_deep_chain():
    p = Pair(2, 0)
    p.merge(0, _chain(1500), t=1)
    p.merge(1, _chain(40)[:3])
    for n in (1, 300, 7):
        p.evict(n, f"chain, {n}")
    p.close()


def test_size_and_eviction_past_unwritten_records():
    """A merge whose rebuilt block does not fit leaves records that no peer holds
    until the next compaction."""
    p = Pair(3, 1)
    seqs = [[7, 2 * i, 1, 2] for i in range(5000)]
    p.f.set_time(2)
    p.o.set_time(2)
    p.f.load_snapshot(1, *pins._csr(seqs))
    p.o.load(1, *pins._csr(seqs))
    p.export(1, "loaded")
    p.f.compact()
    p.merge(0, [[7, 4, 1, 2, 2], [9, 9], [7, 5, 5]])
    assert p.f.info()["merge_refusals"] >= 1, p.f.info()
    for k, n in enumerate((3, 500)):
        p.evict(n, f"past unwritten records, {k}")
    p.export(0, "the inserts")
    p.f.compact()
    p.evict(77, "after a compaction")
    p.close()


@pytest.mark.parametrize("records", [1 << 18, (1 << 18) + 1])
def test_export_order_around_the_bitmap_limit(records):
    """Leaves put in order by a bitmap over the records, and by a sort past it."""
    from paper_2606_17059_amd import Forest
    rng = np.random.default_rng(3)
    pairs = [[a, b] for a in range(512) for b in range(512)][:records - 512]
    mine = [pairs[i] for i in rng.choice(len(pairs), 700, replace=False)]
    f = Forest(2)
    for p, seqs in ((1, pairs), (0, mine)):
        f.load_snapshot(p, *pins._csr(seqs))
    announce(f"export among {records} records")
    t, o = f.export_snapshot(0)
    assert f.info()["num_nodes"] == records
    got = pins.csr_to_list(t.cpu().numpy(), o.cpu().numpy())
    assert sorted(map(tuple, got)) == sorted(map(tuple, mine))
    assert f.tree_tokens(0) == len({tuple(s[:k]) for s in mine for k in (1, 2)})
    f.close()
