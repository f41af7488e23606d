"""Small batches of long queries, which a team of 2 to 16 waves serves each: a
mismatch, an end or an edge at, before and after the ends of the waves' shares,
against the CPU oracle; every width of labels and of peer masks; bad offsets;
and batches one query past the rule's limits."""
import numpy as np
import pytest

import oracle
import pins
from gpu_util import announce, assert_rows_equal, device

pytestmark = pytest.mark.gpu


def _share(n, waves):
    """Tokens a wave takes of a label of n (equal shares in whole lines, at most 1,024)."""
    return min((-(-n // waves) + 31) // 32 * 32, 1024)


def _queries(rng, long, alone, vocab, waves, count):
    """Copies of `long` (labels of len(alone) and len(long) - alone tokens) cut or changed at places."""
    at = {0, 1, 127, 128, 255, 256, 257, 258, alone - 1, alone, alone + 1, len(long) - 1}
    for start, n in ((0, alone), (alone, len(long) - alone)):
        e = _share(n, waves)
        for w in {1, 2, waves - 1, waves, waves + 1}:
            at |= {start + w * e + k for k in (-1, 0, 1)}
    at = sorted(x for x in at if 0 <= x < len(long))
    out = [long, long + [5], []]
    for x in at:
        out.append(long[:x] + [(long[x] + 1) % vocab] + long[x + 1:])
        if len(out) % 3 == 0:
            out.append(long[:x])
    rng.shuffle(out)
    return out[:count]


@pytest.mark.parametrize("P, vocab, mean, waves", [
    (3, 30000, 1100, 2), (130, 120000, 2500, 4), (70, 1 << 30, 5000, 8), (1000, 60000, 9000, 16), (300, 70000, 33000, 16),
    (513, 100000, 1800, 2),
])
@pytest.mark.parametrize("prefix", [0, 1, 300])
def test_team_rows(P, vocab, mean, waves, prefix):
    import torch
    from paper_2606_17059_amd import Forest
    rng = np.random.default_rng(P + prefix)
    shared = rng.integers(0, vocab, prefix).tolist()  # 0: the root has several children
    long = shared + rng.integers(0, vocab, mean * 2).tolist()
    alone = prefix + mean // 3 + 1  # another sequence leaves the long one here
    other = long[:alone] + [(long[alone] + 1) % vocab] + rng.integers(0, vocab, 90).tolist()
    f, o = Forest(P), oracle.Oracle(P)
    for p, seqs in ((0, [long]), (P - 1, [other, shared + [7, 8]]), (P // 2, [long[:alone + 700], [9, 9]])):
        t, off = pins._csr(seqs)
        f.load_snapshot(p, t, off)
        o.load(p, t, off)
    qs = _queries(rng, long, alone, vocab, waves, 60)
    t, off = pins._csr(qs)
    assert 1024 * waves // 2 <= len(t) // len(qs)  # the rule gives at least this many waves
    announce(f"team route P={P} mean={len(t) // len(qs)} waves>={waves}")
    qt, qo = torch.from_numpy(t).to(device()), torch.from_numpy(off).to(device())
    m, c = f.route(qt, qo)
    mo, co = o.route(t, off, 4)
    assert_rows_equal(m.cpu().numpy(), c.cpu().numpy(), mo, co, what="team")
    # the selection instances, and the same rows from them
    ms, best, second = f.route_select(qt, qo, None, P - 1, False)
    assert np.array_equal(ms.cpu().numpy(), mo) and np.array_equal(best.cpu().numpy(), co)
    key = mo.astype(np.int64) * (2 * P) + (P - np.arange(P))
    key[np.arange(len(qs)), co] = -1
    assert np.array_equal(second.cpu().numpy(), key.argmax(axis=1).astype(np.int32))
    # offsets outside the tokens: -1 in that row only
    bad = off.copy()
    bad[-1] = len(t) + 5
    m2, c2 = f.route(qt, torch.from_numpy(bad).to(device()))
    assert (m2[-1] == -1).all() and int(c2[-1]) == -1
    assert torch.equal(m2[:-1], m[:-1]) and torch.equal(c2[:-1], c[:-1])
    f.close()


@pytest.mark.parametrize("n, mean", [(512, 1023), (512, 1024), (513, 1024), (1024, 2048), (1025, 2048), (2048, 4096),
                                     (2049, 4100)])
def test_team_limits(n, mean):
    import torch
    from paper_2606_17059_amd import Forest
    rng = np.random.default_rng(n)
    stem = rng.integers(0, 50000, mean).astype(np.int32)
    f = Forest(2)
    half = stem[:mean // 2]
    for p, s in ((0, stem), (1, half)):
        off = np.array([0, len(s)], np.int64)
        f.load_snapshot(p, s, off)
    q = np.tile(stem, (n, 1))
    at = rng.integers(0, mean, n)
    q[np.arange(n), at] += 1
    off = np.arange(n + 1, dtype=np.int64) * mean
    announce(f"team limits n={n} mean={mean}")
    m, c = f.route(torch.from_numpy(q.reshape(-1)).to(device()), torch.from_numpy(off).to(device()))
    mo = np.stack([at, np.minimum(at, mean // 2)], 1).astype(np.int32)
    co = mo.argmax(axis=1).astype(np.int32)
    assert_rows_equal(m.cpu().numpy(), c.cpu().numpy(), mo, co, what="limits")
    f.close()


@pytest.mark.parametrize("P", [3, 130, 1000])
@pytest.mark.parametrize("n", [1, 48, 512, 2048])
def test_batch_in_a_larger_buffer(n, P):
    """Queries of 0 to 5,000 tokens at the start of a buffer of 4 M, as a server's
    staging buffer: teams are launched by the buffer's size, and every query ends the
    waves its own length does not pay for (at 1,023 and 1,024 tokens, 2,047 and 2,048
    and so on), some of a batch all but one."""
    import torch
    from paper_2606_17059_amd import Forest
    rng = np.random.default_rng(n + P)
    f, o = Forest(P), oracle.RadixOracle(P)
    stems = [rng.integers(0, 70000, 5200).tolist() for _ in range(4)]
    for p in {0, P // 2, P - 1}:
        seqs = [s[:int(rng.integers(400, 5200))] for s in stems] + [stems[p % 4][:700] + [p] * 300]
        t, off = pins._csr(seqs)
        f.load_snapshot(p, t, off)
        o.load(p, t, off)
    edges = [0, 1, 256, 257, 511, 512, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 5000]
    qs = []
    for i in range(n):
        L = edges[(i + n) % len(edges)] if i % 2 == 0 else int(rng.integers(0, 5000))
        q = stems[int(rng.integers(0, 4))][:L]
        if q and rng.random() < 0.5:
            at = int(rng.integers(0, L))
            q = q[:at] + [q[at] + 1] + q[at + 1:]
        qs.append(q)
    t, off = pins._csr(qs)
    buf = np.full(max(4 << 20, len(t) + 9), 7, np.int32)
    buf[:len(t)] = t
    announce(f"{n} queries of {P} peers in a larger buffer")
    m, c = f.route(torch.from_numpy(buf).to(device()), torch.from_numpy(off).to(device()))
    mo, co = o.route(t, off, 8)
    assert_rows_equal(m.cpu().numpy(), c.cpu().numpy(), mo, co, what="larger buffer")
    f.close()
    o.close()


@pytest.mark.parametrize("P", [64, 65, 512, 513])
@pytest.mark.parametrize("n", [5, 256, 257])
@pytest.mark.parametrize("mean", [1023, 1024, 2047, 2048, 5119, 5120, 8191, 8192])
def test_team_limits_by_mask_words(P, n, mean):
    """The shortest mean a team serves depends on the mask words of a record: 1,024
    tokens with one, 2,048 with two to eight, 5,120 (8,192 past 256 queries) with sixteen."""
    import torch
    from paper_2606_17059_amd import Forest
    rng = np.random.default_rng(P + n + mean)
    stem = rng.integers(0, 50000, mean).astype(np.int32)
    f = Forest(P)
    for p, s in ((0, stem), (P - 1, stem[:mean // 2])):
        f.load_snapshot(p, s, np.array([0, len(s)], np.int64))
    q = np.tile(stem, (n, 1))
    at = rng.integers(0, mean, n)
    q[np.arange(n), at] += 1
    announce(f"team limits P={P} n={n} mean={mean}")
    m, c = f.route(torch.from_numpy(q.reshape(-1)).to(device()),
                   torch.from_numpy(np.arange(n + 1, dtype=np.int64) * mean).to(device()))
    mo = np.zeros((n, P), np.int32)
    mo[:, 0] = at
    mo[:, P - 1] = np.minimum(at, mean // 2)
    assert_rows_equal(m.cpu().numpy(), c.cpu().numpy(), mo, mo.argmax(axis=1).astype(np.int32), what="limits")
    f.close()
