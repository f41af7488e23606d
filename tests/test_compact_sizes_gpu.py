"""Compaction at the sizes where its launches change: one workgroup up to 8,192
records, levels in batches past that (chains deeper than a batch of levels), a
label pool over what one wait serves, separators past both levels, mask words
past the first; several in a row, which reuse the arrays of the one before."""
import numpy as np
import pytest

import pins
import workloads as W
from gpu_util import announce, assert_rows_equal, device, gpu_route

pytestmark = pytest.mark.gpu


def _merge(f, o, peers, seqs):
    import torch
    t, off = pins._csr(seqs)
    peers = np.asarray(peers, np.int32)
    f.merge(*[torch.from_numpy(x).to(device()) for x in (peers, t, off)])
    o.merge(peers, t, off)


def _wide(n):
    return [[7, 2 * i, 5, i % 3] for i in range(n)]


CASES = {
    "8192 records": lambda rng: _wide(8190),  # the root, [7] and one per child
    "8193 records": lambda rng: _wide(8191),
    "chain of 40 over 9000": lambda rng: _wide(9000) + [[3, 1, 4, 1, 5][:i % 6] + list(range(i)) for i in range(1, 41)],
    "small and deep": lambda rng: [list(range(i)) for i in range(1, 400)],
    "labels over one wait's bound": lambda rng: [[i] + rng.integers(0, 90000, 30000).tolist() for i in range(150)],
    "second-level separators": lambda rng: _wide(4200) + [[8, i] for i in range(65)] + [[9, i] for i in range(64)],
}


@pytest.mark.parametrize("what", list(CASES))
@pytest.mark.parametrize("P", [2, 130])
def test_compaction_sizes(what, P):
    import oracle
    from paper_2606_17059_amd import Forest
    rng = np.random.default_rng(17)
    f, o = Forest(P), oracle.RadixOracle(P)
    seqs = CASES[what](rng)
    _merge(f, o, rng.integers(0, P, len(seqs)), seqs)
    queries = [s[:400] for s in seqs[::max(1, len(seqs) // 700)]] + [s[:-1] + [99999] for s in seqs[:50]]
    qt, qo = pins._csr(queries)
    bits = 17 if max(max(s) for s in seqs) > 65535 else 16
    for k in range(4):
        announce(f"compaction {k} of {what}, {P} peers")
        before, after = f.compact()
        info = f.info()
        assert info["num_nodes"] == after <= before and info["label_bits"] == bits
        m, c = gpu_route(f, W.SeqSet(qt, qo, None), f"{what} {k}")
        m_or, c_or = o.route(qt, qo, 8)
        assert_rows_equal(m, c, m_or, c_or, what=f"{what} {k}")
        more = [s[:len(s) // 2] + [50 + k, i % 5] for i, s in enumerate(seqs[k::97])] + [[k + 1]]
        if k < 2:
            _merge(f, o, rng.integers(0, P, len(more)), more)
        else:
            assert f.compact() == (after, after)  # nothing left to drop
        t, off = pins._csr(more)
        m, c = gpu_route(f, W.SeqSet(t, off, None), f"{what} {k} merged")
        m_or, c_or = o.route(t, off, 8)
        assert_rows_equal(m, c, m_or, c_or, what=f"{what} {k} merged")
    f.close()
    o.close()
