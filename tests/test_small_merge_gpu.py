"""Merges and touches of at most 64 sequences (one launch) and just above
(rounds of launches), against the CPU oracles: conflicts on slots and edges
inside a batch, wide parents past the one launch's limit, growth, token widths,
mask words past the first."""
import numpy as np
import pytest

import pins
import workloads as W
from gpu_util import announce, assert_rows_equal, device, gpu_route, oracle_for

pytestmark = pytest.mark.gpu


def _dev(peers, seqs):
    import torch
    t, o = pins._csr(seqs)
    return [torch.from_numpy(x).to(device()) for x in (np.asarray(peers, np.int32), t, o)]


def _check(f, o, queries, what):
    t, off = pins._csr(queries)
    m, c = gpu_route(f, W.SeqSet(t, off, None), what)
    m_or, c_or = o.route(t, off, 4)
    assert_rows_equal(m, c, m_or, c_or, what=what)


def _seqs(rng, vocab, k, lo=0, hi=14, known=()):
    """Random sequences, many of them grown from the start of a known one."""
    out = []
    for _ in range(k):
        s = list(known[int(rng.integers(0, len(known)))]) if len(known) and rng.random() < 0.6 else []
        s = s[:int(rng.integers(0, len(s) + 1))]
        out.append(s + rng.integers(0, vocab, int(rng.integers(lo, hi))).tolist())
    return out


@pytest.mark.parametrize("n", [1, 2, 17, 63, 64, 65])
@pytest.mark.parametrize("P", [3, 130])
def test_batches_around_one_lane_each(n, P):
    """Batches of n conflicting inserts (shared slots, shared edges, chains of
    cuts, duplicates, empty sequences, bad peers), then every stored sequence
    and random ones routed."""
    import oracle
    from paper_2606_17059_amd import Forest, RouterError
    rng = np.random.default_rng(100 * n + P)
    f, o = Forest(P), oracle.Oracle(P)
    known = [[]]
    for step in range(6):
        vocab = [2, 3, 8, 2, 100, 3][step]
        seqs = _seqs(rng, vocab, n, known=known)
        peers = rng.integers(0, P, n)
        if step == 2 and n > 2:
            seqs[1:] = [seqs[0][:i % (len(seqs[0]) + 1)] for i in range(1, n)]  # every cut of one path
        bad = np.array(peers)
        bad[0] = P if step == 4 else bad[0]
        announce(f"small merge n={n} P={P} step={step}")
        f.merge(*_dev(bad, seqs))
        keep = [i for i in range(n) if 0 <= bad[i] < P]
        t, off = pins._csr([seqs[i] for i in keep])
        o.merge(np.asarray([bad[i] for i in keep], np.int32), t, off)
        if step == 4:
            with pytest.raises(RouterError, match="1 device inputs were skipped"):
                f.check()
        known += [seqs[i] for i in keep if seqs[i]]
        _check(f, o, known[-200:] + _seqs(rng, vocab, 60, known=known), f"n={n} P={P} step={step}")
    f.check()
    f.close()
    o.close()


def test_wide_parent_and_growth():
    """A root of 17,000 children has more chunks than the one launch moves; an
    insert there and one elsewhere in the same batch, then a leaf of 200,000
    tokens, which outgrows the pool."""
    import oracle
    from paper_2606_17059_amd import Forest
    f, o = Forest(2), oracle.RadixOracle(2)
    wide = [[2 * i, 5] for i in range(17000)]
    t, off = pins._csr(wide)
    f.load_snapshot(0, t, off)
    o.load(0, t, off)
    rng = np.random.default_rng(4)
    for step, seqs in enumerate([[[6, 5, 1], [7, 1]], [[6, 5, 2, 9]], [[3, 3], [6, 5, 2, 8], [4, 4]],
                                 [[8] + rng.integers(0, 60000, 200000).tolist()], [[8, 8], [9], [10, 5, 7]]]):
        announce(f"wide parent, step {step}")
        f.merge(*_dev([1] * len(seqs), seqs))
        t, off = pins._csr(seqs)
        o.merge(np.full(len(seqs), 1, np.int32), t, off)
        queries = [s[:500] for s in seqs] + [s[:-1] for s in seqs] + wide[::170] + [[2 * i + 1, 5] for i in range(20)]
        _check(f, o, queries, f"wide parent, step {step}")
    f.close()
    o.close()


def test_narrow_copy_of_every_alignment():
    """One-launch merges write the narrow labels as they go: 17-bit sequences
    of 1 to 200 tokens end to end in the pool, queried with bit 16 flipped at
    each kind of place; then a token past 17 bits."""
    import oracle
    from paper_2606_17059_amd import Forest
    rng = np.random.default_rng(8)
    f, o = Forest(3), oracle.Oracle(3)
    f.merge(*_dev([0], [[1, 2, 3]]))
    o.merge(np.zeros(1, np.int32), *pins._csr([[1, 2, 3]]))
    assert f.info()["label_bits"] == 16
    stored = []
    for step in range(6):
        seqs = [[100 * step + L] + (rng.integers(0, 2, L) * 65536 + rng.integers(0, 3, L)).tolist()
                for L in range(step + 1, 200, 11)]
        peers = rng.integers(0, 3, len(seqs))
        announce(f"17-bit one-launch merge {step}")
        f.merge(*_dev(peers, seqs))
        o.merge(peers.astype(np.int32), *pins._csr(seqs))
        stored += seqs
        flips = []
        for s in stored[-18:]:
            for at in {1, len(s) // 2, len(s) - 1}:
                flips.append(s[:at] + [s[at] ^ 65536] + s[at + 1:])
        _check(f, o, stored + flips, f"17-bit merge {step}")
    assert f.info()["label_bits"] == 17
    f.merge(*_dev([1], [[1, 2, 200000]]))
    o.merge(np.ones(1, np.int32), *pins._csr([[1, 2, 200000]]))
    assert f.info()["label_bits"] == 32
    _check(f, o, stored + [[1, 2, 200000, 4], [1, 2, 200000 - 131072]], "after a wide token")
    f.close()
    o.close()


@pytest.mark.parametrize("n", [1, 5, 64, 65, 300])
def test_touches_then_evictions(n):
    """Touches of n queries (empty, past the tree, ending inside labels, with
    bad offsets) at rising times; evictions then take paths in the oracle's
    order, and other peers keep theirs."""
    import oracle
    import torch
    from paper_2606_17059_amd import Forest
    rng = np.random.default_rng(n)
    P, L = 70, 66
    f, o = Forest(P), oracle.Oracle(P)
    f.set_local_peer(L)
    o.set_local(L)
    base = _seqs(rng, 3, 60, 1, 12)
    peers = np.where(np.arange(60) % 3 == 0, L, rng.integers(0, P, 60)).astype(np.int32)
    f.merge(*_dev(peers, base))
    o.merge(peers, *pins._csr(base))
    for step in range(4):
        f.set_time(step + 1)
        o.set_time(step + 1)
        qs = _seqs(rng, 3, n, 0, 6, known=base)
        t, off = pins._csr(qs)
        dt, do = torch.from_numpy(t).to(device()), torch.from_numpy(off).to(device())
        if step == 1:
            # the last query's end lies past the batch: ignored, and not counted as skipped
            do[-1] += 1000
            qs = qs[:-1]
        announce(f"touch n={n} step={step}")
        f.touch(dt, do)
        if qs:
            o.touch(*pins._csr(qs))
        f.check()
        k = int(rng.integers(1, 9))
        assert f.evict_lru(k) == o.evict(k), (n, step)
        et, eo = f.export_snapshot(L)
        got = sorted(map(tuple, pins.csr_to_list(et.cpu().numpy(), eo.cpu().numpy())))
        assert got == sorted(map(tuple, pins.csr_to_list(*o.export(L)))), (n, step)
        _check(f, o, base + qs, f"touch n={n} step={step}")
    f.close()
    o.close()


def _long_heads(rng, n, L):
    """n sequences of L tokens: half of them grow from the other half's middles."""
    own = rng.integers(0, 60000, (n, L))
    own[:, 0] = np.arange(n) * 5 + 10
    for i in range(1, n, 2):
        own[i, :L // (1 + i % 3)] = own[i - 1, :L // (1 + i % 3)]
    return own.tolist()


@pytest.mark.parametrize("n,L,launches", [(16, 20000, False), (17, 19000, False), (17, 21000, True), (64, 1300, False),
                                          (64, 1400, True), (64, 8000, True)])
def test_long_sequences_are_left_to_the_launches(n, L, launches):
    """Past 16 sequences, batches whose sequences times valid tokens pass 5.5 million go to
    the rounds of launches, which take scratch; the forest has room for either.  A bad
    entry is counted once.  Touches stay in one launch."""
    import oracle
    from paper_2606_17059_amd import Forest, RouterError
    rng = np.random.default_rng(n + L)
    f, o = Forest(3), oracle.RadixOracle(3)
    room = [[1, 2, 3]] + [[9, i] + rng.integers(0, 100, 40000).tolist() for i in range(90)]
    t, off = pins._csr(room)
    f.load_snapshot(2, t, off)
    o.load(2, t, off)
    queries = [[1, 2, 3, 4]]
    _check(f, o, queries, "upload")
    before = f.info()["device_bytes"]
    seqs = _long_heads(rng, n, L)
    peers = rng.integers(0, 3, n)
    bad = np.array(peers)
    bad[n // 2] = 3
    announce(f"{n} sequences of {L} tokens")
    f.merge(*_dev(bad, seqs))
    assert (f.info()["device_bytes"] > before) == launches, (before, f.info())
    with pytest.raises(RouterError, match="1 device inputs were skipped"):
        f.check()
    keep = [i for i in range(n) if i != n // 2]
    t, off = pins._csr([seqs[i] for i in keep])
    o.merge(peers[keep].astype(np.int32), t, off)
    queries += seqs + [s[:L // 2] + [-5] for s in seqs]
    _check(f, o, queries, f"{n} of {L}")
    f.set_local_peer(1)
    held = f.info()["device_bytes"]
    t, off = pins._csr([s[:L - 3] for s in seqs])
    import torch
    announce(f"touch of {n} sequences of {L} tokens")
    f.touch(*[torch.from_numpy(x).to(device()) for x in (t, off)])
    assert f.info()["device_bytes"] == held
    _check(f, o, queries, f"{n} of {L}, touched")
    f.check()
    f.close()
    o.close()


def test_small_batch_outgrows_the_pool_between_rounds():
    """Twelve sequences that part from each other one after the other, their tails
    more than the pool has left: the first rounds' tails fit, a later round's do not,
    and the launches take over with some of the batch in."""
    import oracle
    from paper_2606_17059_amd import Forest
    rng = np.random.default_rng(12)
    f, o = Forest(2), oracle.RadixOracle(2)
    f.merge(*_dev([0], [[5, 5]]))
    o.merge(np.zeros(1, np.int32), *pins._csr([[5, 5]]))
    path = rng.integers(0, 50, 40).tolist()
    order = rng.permutation(12)
    seqs = [path[:3 * k + 2] + [100 + k] + rng.integers(0, 30000, 40000).tolist() for k in order]
    peers = np.arange(12) % 2
    announce("12 tails of 40,000 tokens into a pool of 262,144")
    f.merge(*_dev(peers, seqs))
    o.merge(peers.astype(np.int32), *pins._csr(seqs))
    queries = seqs + [s[:500] for s in seqs] + [path[:k] for k in range(40)] + [[5, 5, 5]]
    _check(f, o, queries, "outgrown")
    assert f.info()["pool_tokens"] <= 262144 + sum(map(len, seqs))
    f.check()
    f.close()
    o.close()


@pytest.mark.parametrize("n", [64, 65, 75, 200])
@pytest.mark.parametrize("order", ["shortest first", "longest first", "shuffled"])
def test_chains_hand_over_from_launch_to_launch(n, order):
    """A chain of inserts that part from one new path a token after another.  With the
    shortest first a round places one of them, the next cut of what the last one hung:
    up to 64 are done in one launch, 75 leave few enough for it after the queued
    rounds, 200 pass to the host's rounds; the other orders take fewer."""
    import oracle
    from paper_2606_17059_amd import Forest
    rng = np.random.default_rng(n)
    f, o = Forest(3), oracle.RadixOracle(3)
    stored = []
    for k in range(2):  # the second chain with as many rounds queued as the first took
        path = [500 + k] + rng.integers(0, 40, n).tolist()
        seqs = [path[:i + 1] + [100 + i, 1, 2] for i in range(n)]
        if order != "shortest first":
            seqs = seqs[::-1] if order == "longest first" else [seqs[i] for i in rng.permutation(n)]
        peers = rng.integers(0, 3, n)
        announce(f"chain {k} of {n}, {order}")
        f.merge(*_dev(peers, seqs))
        o.merge(peers.astype(np.int32), *pins._csr(seqs))
        stored += seqs
        _check(f, o, stored + [s[:-2] + [9] for s in stored] + [path[:i] for i in range(0, n, 7)], f"chain {k}")
    assert f.tree_tokens(1) == len({tuple(s[:i]) for p, s in _held(f, 1) for i in range(1, len(s) + 1)})
    f.check()
    f.close()
    o.close()


def _held(f, p):
    t, o = f.export_snapshot(p)
    return [(p, s) for s in pins.csr_to_list(t.cpu().numpy(), o.cpu().numpy())]
