"""Merges that run out of device capacity: what they ask for, and what they leave."""
import numpy as np
import pytest

import pins
import workloads as W
from gpu_util import announce, assert_rows_equal, device, gpu_route

pytestmark = pytest.mark.gpu


def _merge(f, o, peers, seqs, what):
    import torch
    t, off = pins._csr(seqs)
    peers = np.asarray(peers, np.int32)
    announce(what)
    f.merge(*[torch.from_numpy(x).to(device()) for x in (peers, t, off)])
    o.merge(peers, t, off)


def _check(f, o, queries, what):
    t, off = pins._csr(queries)
    m, c = gpu_route(f, W.SeqSet(t, off, None), what)
    m_or, c_or = o.route(t, off, 8)
    assert_rows_equal(m, c, m_or, c_or, what=what)


def _capacity_bytes(info, pool, records):
    """Device bytes of `pool` label tokens (int32, the 16-bit copy and its bit plane) and `records` records."""
    return pool * 4 + pool * 2 + pool // 8 + records * (32 + 4 + 4 + 8 * info["mask_words"])


def test_rounds_queued_behind_a_refusal_ask_for_nothing():
    """Chains of cuts teach the forest to queue four rounds; then a batch outgrows
    its pool, of 262,144 tokens, in the first of them.  The pool that the forest
    grows to holds the batch once (not once for every queued round), and one
    round's records stay unwritten."""
    import oracle
    from paper_2606_17059_amd import Forest
    rng = np.random.default_rng(6)
    P = 3
    f, o = Forest(P), oracle.RadixOracle(P)
    stored = []
    for k in range(2):
        path = rng.integers(0, 50, 200).tolist()
        seqs = [[1000 + k] + path[:i] + [60 + i] for i in rng.permutation(200)]
        _merge(f, o, rng.integers(0, P, 200), seqs, f"chain {k}")
        stored += seqs
    before = f.info()
    assert before["merge_refusals"] == 0
    n, L = 300, 4000
    seqs = [[2000 + i] + rng.integers(0, 30000, L - 1).tolist() for i in range(n)]
    _merge(f, o, rng.integers(0, P, n), seqs, "past the pool")
    info = f.info()
    assert info["merge_refusals"] == 1
    # the refused round's and the repeated one's: the root's block with the new leaves
    block = 2 + n
    assert info["num_nodes"] <= before["num_nodes"] + 2 * block, (before, info)
    need = 262144 + n * L
    assert info["pool_tokens"] <= need
    grown = info["device_bytes"] - before["device_bytes"] + _capacity_bytes(info, 262144, 0)
    assert grown <= _capacity_bytes(info, need + 64, 0) + (1 << 20), (before, info)
    _check(f, o, stored + [s[:400] for s in seqs] + [s[:-1] + [7] for s in seqs[:20]], "after the refusal")
    f.check()
    f.close()
    o.close()


@pytest.mark.parametrize("n,L", [(100, 20000), (500, 1200)])
@pytest.mark.parametrize("load", [True, False])
def test_first_batch_past_the_pool_is_sized_before_it_runs(n, L, load):
    """A cold forest's first snapshot or merge does not fit the pool it starts
    with (262,144 tokens): the pool grows to what the walk finds missing, nothing
    is refused, and the records hold the batch without gaps."""
    import oracle
    import torch
    from paper_2606_17059_amd import Forest
    rng = np.random.default_rng(n)
    f, o = Forest(2), oracle.RadixOracle(2)
    heads = rng.integers(0, 30000, (8, L // 2))
    seqs = [heads[i % 8].tolist() + rng.integers(0, 30000, L - L // 2).tolist() for i in range(n)]
    t, off = pins._csr(seqs)
    if load:
        announce(f"cold load {n} x {L}")
        f.load_snapshot_device(1, *[torch.from_numpy(x).to(device()) for x in (t, off)])
        o.merge(np.ones(n, np.int32), t, off)
    else:
        _merge(f, o, np.ones(n), seqs, f"cold merge {n} x {L}")
    info = f.info()
    assert info["merge_refusals"] == 0
    assert info["pool_tokens"] <= n * L
    assert info["device_bytes"] <= _capacity_bytes(info, n * L + 64, 0) + (8 << 20), info
    _check(f, o, [s[:L - i] for i, s in enumerate(seqs[:64])] + [s[:L // 2] + [-1] for s in seqs[::9]], "cold")
    f.close()
    o.close()
