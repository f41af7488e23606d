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
    rt.on["small_merge_kernel"] = rt.small_merge(dict(add_nodes=65, add_pool=added))
    assert f.merge(65) == 0
    return f


@pytest.mark.parametrize("what", ["merge", "touch"])
def test_room_for_a_merge_like_the_last_one_is_not_a_condition(rt, what):
    """A merge wants as much spare room as the last ones took.  Where the ids or
    the memory do not allow that, it runs in the room there is."""
    for added, free in ((3 << 30, None), (1 << 20, 1 << 16)):
        f = rt.forest(2)
        f.close()
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
