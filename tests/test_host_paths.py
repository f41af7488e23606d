"""The library's host code without a GPU: what it allocates, which launches it
chooses, and what it does when memory or ids run out (tests/host_runtime.py)."""
import pytest

import host_runtime


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return host_runtime.build(tmp_path_factory.mktemp("host_paths"))


@pytest.fixture
def rt(so, monkeypatch):
    return host_runtime.HostRuntime(so, monkeypatch)


def test_forest_on_the_host_runtime(rt):
    f = rt.forest(3, [[[1, 2, 3]], [[1, 2], [4]]])
    assert f.merge(2) == 0 and f.info().num_nodes == 4
    assert rt.launched("small_merge_kernel") == 1
    f.close()
    assert rt.used() == 0


def _after_a_large_merge(rt, added):
    """A forest whose last merge of 65 sequences added that many label tokens."""
    f = rt.forest(2, [[[1, 2, 3]]])
    rt.large_merge(f, 5000, added)
    return f


@pytest.mark.parametrize("what", ["merge", "touch"])
def test_room_for_a_merge_like_the_last_one_is_not_a_condition(rt, what):
    """A merge wants as much spare room as the last ones took.  Where the ids or
    the memory do not allow that, it runs in the room there is."""
    for added, free in ((3 << 30, None), (1 << 20, 1 << 16)):
        f = _after_a_large_merge(rt, added)
        if what == "touch":
            assert f.L.pr_set_local_peer(f.h, 0) == 0
        if free is not None:
            rt.limit(rt.used() + free)
        assert getattr(f, what)(65) == 0, (added, f.error())
        assert getattr(f, what)(65) == 0
        rt.limit(None)
        f.close()


def test_a_touch_reserves_no_label_tokens(rt):
    f = _after_a_large_merge(rt, 200000)  # of the 262,144 the pool starts with
    assert f.L.pr_set_local_peer(f.h, 0) == 0
    before = f.info()
    assert f.touch(65) == 0
    assert f.info().layout_epoch == before.layout_epoch and f.info().device_bytes == before.device_bytes
    f.close()


def test_a_refusal_is_met_exactly_where_memory_is_short(rt):
    """Growth is fourfold where there is memory for it, else to what is needed."""
    f = rt.forest(2, [[[1, 2, 3]]])
    rt.large_merge(f, 1 << 18, 100)
    rt.on["small_merge_kernel"] = rt.small_merge(dict(done=0, overflow=1, add_nodes=(1 << 18) + (1 << 17)))
    rt.limit(rt.used() + 49_000_000)  # for the records asked for, not for four times those there are
    status, error = f.merge(65), f.error()
    rt.limit(None)
    f.close()
    assert status == 0, error


def test_a_refusal_the_memory_cannot_meet_is_an_error(rt):
    """A refused round's records are a condition: without memory for them the
    merge fails and the forest refuses what follows."""
    f = rt.forest(2, [[[1, 2, 3]]])
    assert f.merge(65) == 0
    rt.on["small_merge_kernel"] = rt.small_merge(dict(done=0, overflow=1, add_nodes=1 << 24))
    rt.limit(rt.used() + (1 << 16))
    assert f.merge(65) == rt.R.PR_ENOMEM
    assert f.merge(65) == rt.R.PR_ESTATE
    rt.limit(None)
    f.close()


def _rounds(rt, call):
    rt.clear()
    assert call() == 0
    return rt.launched("merge_walk_kernel")


def test_rounds_queued_follow_the_batches_of_their_kind(rt):
    """As many rounds as the last batch of the kind took: merges, snapshots and
    touches each have their own count, and a refused batch says nothing."""
    f = rt.forest(2, [[[1, 2, 3]]])
    assert f.merge(65) == 0 and f.L.pr_set_local_peer(f.h, 0) == 0
    rt.on["small_merge_kernel"] = rt.small_merge(rounds=3)
    assert f.merge(65) == 0
    rt.on["small_merge_kernel"] = rt.small_merge(rounds=1)
    assert _rounds(rt, lambda: f.touch(65)) == 2  # none seen so far
    assert _rounds(rt, lambda: f.touch(65)) == 1
    load = lambda: f.load_device(1, 65)  # noqa: E731
    assert _rounds(rt, load) == 2
    assert _rounds(rt, load) == 1
    # refused at its first of three queued rounds; the host-driven ones find all done
    rt.on["small_merge_kernel"] = rt.small_merge(dict(done=0, overflow=1, rounds=1, add_nodes=10), rounds=3)
    assert _rounds(rt, lambda: f.merge(65)) == 3 + 1
    assert _rounds(rt, lambda: f.merge(65)) == 3
    f.close()


def _with_spare(rt, records=20000, pool=1 << 18):
    """A forest whose last compaction kept the arrays it replaced, with merge scratch
    for 3,000 sequences and a sort's for 1,600."""
    f = rt.forest(2, [[[1, 2, 3]]])
    rt.large_merge(f, records, pool)
    assert [f.merge(n) for n in (1500, 1600)] == [0, 0]
    rt.compacts_to(records, pool)
    assert f.L.pr_set_local_peer(f.h, 0) == 0
    rt.walk_finds(nodes=10, leaves=10)
    assert f.compact() == 0 and f.export(1)[0] == 0
    return f


@pytest.mark.parametrize("what", ["eviction", "merge", "export"])
def test_what_a_compaction_kept_is_given_back_when_memory_runs_out(rt, what):
    """The arrays a compaction keeps for the next one make room for any later
    call's scratch: it succeeds as it would have without them."""
    f = _with_spare(rt)
    kept = f.info().device_bytes
    rt.walk_finds(nodes=10000, leaves=10000)
    rt.limit(rt.used() + (1 << 10))
    call = {"eviction": lambda: f.evict(5)[0], "merge": lambda: f.merge(3000), "export": lambda: f.export(1)[0]}[what]
    refused, status = rt.refused(), call()
    gone, after = rt.refused() - refused, f.info().device_bytes
    rt.limit(None)
    f.close()
    assert status == 0 and gone == 1 and after < kept  # refused once, beside the kept arrays
    assert rt.used() == 0


def test_room_for_later_merges_is_not_a_condition_of_a_compaction(rt):
    """A compaction leaves room for merges like the recent ones where there is
    memory for it; else it takes what the forest needs."""
    f = rt.forest(2, [[[1, 2, 3]]])
    n = 1 << 20
    rt.large_merge(f, n, 1 << 22)
    rt.walk_finds(nodes=1)
    assert f.export(1)[0] == 0  # its scratch is a compaction's
    rt.compacts_to(n, 1 << 22)
    # the forest once more, with an eighth to spare (48 bytes a record, six a token), not with two such merges on top
    rt.limit(rt.used() + (n * 48 + (1 << 22) * 6) * 10 // 8)
    status = f.compact()
    rt.limit(None)
    f.close()
    assert status == 0


@pytest.mark.parametrize("size", [1, 16])
@pytest.mark.parametrize("left", [1.0, 0.6, 0.4, 0.1])
def test_a_compaction_gives_back_what_it_freed(rt, left, size):
    """A compaction that leaves more than half of the forest keeps the replaced
    arrays, and the next one allocates nothing; one that leaves less of a forest of
    more than 64 MB gives them back, and the image is sized to what is left."""
    f = rt.forest(2, [[[1, 2, 3]]])
    nodes, pool = size << 16, size << 21  # 16 MB, 256 MB
    rt.large_merge(f, nodes, pool)
    for _ in range(100):  # merges since then were small ones
        assert f.merge(65) == 0
    rt.walk_finds(nodes=1)
    assert f.export(1)[0] == 0
    rt.compacts_to(nodes, pool)
    assert f.compact() == 0 and f.compact() == 0
    full = f.info().device_bytes
    rt.compacts_to(int(nodes * left), int(pool * left))
    assert f.compact() == 0
    info = f.info()
    assert info.num_nodes == int(nodes * left)
    if left > 0.5 or size == 1:
        rt.limit(rt.used())
        refused, status = rt.refused(), f.compact()
        rt.limit(None)
        assert status == 0 and rt.refused() == refused
    else:
        # records once more sized by the old forest's, tokens by what is left; room for the recent merges
        assert info.device_bytes <= full / 2
        image = 48 * nodes * 5 / 4 + 6.2 * pool * left * 5 / 4
        assert info.device_bytes <= image + 2 * 6.2 * pool / 16 + 2 * 48 * nodes / 16 + (12 << 20)
    f.close()
    assert rt.used() == 0


def test_sizes_and_evictions_after_a_refusal(rt):
    """A refused round leaves no record unwritten, so sizes and evictions go on
    taking the passes over the records."""
    f = rt.forest(2, [[[1, 2, 3]]])
    assert f.merge(65) == 0 and f.L.pr_set_local_peer(f.h, 0) == 0
    rt.on["small_merge_kernel"] = rt.small_merge(dict(done=0, overflow=1, add_nodes=500))
    assert f.merge(65) == 0 and f.info().merge_refusals == 1
    rt.size_is(42)
    rt.clear()
    assert f.tokens(0) == (0, 42)
    rt.on["evict_kernel"] = rt.evicts(7)
    assert f.evict(7) == (0, 7)
    assert rt.launched("tree_walk_kernel") == 0 and rt.launched("evict_kernelILb1E") == 1, rt.launches
    f.close()


@pytest.mark.parametrize("records,walks", [(1 << 23, 0), ((1 << 23) + 1, 1)])
def test_a_tree_among_very_many_records_is_walked(rt, records, walks):
    """The pass over all records is not taken for a tree that a walk finds sooner;
    trees too large for the walk take it all the same."""
    f = rt.forest(2, [[[1, 2, 3]]])
    rt.large_merge(f, records, 100)
    rt.size_is(42)
    rt.walk_counts(42)
    rt.clear()
    assert f.tokens(0) == (0, 42)
    assert (rt.launched("tree_walk_kernel"), rt.launched("tree_size_kernel")) == (walks, 1 - walks)
    rt.walk_finds(nodes=5)
    rt.clear()
    assert f.tokens(1) == (0, 42)
    assert (rt.launched("tree_walk_kernel"), rt.launched("tree_size_kernel")) == (walks, 1)
    f.close()
