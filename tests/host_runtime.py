"""The library's host code on a HIP runtime without a GPU (tests/c/host_runtime.cpp).

`HostRuntime` links the library's objects with that runtime and answers kernel
launches: the few whose results the host reads have a plain default below, which a
test overrides by the kernel's name."""
from __future__ import annotations

import ctypes
import os
import re
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

_vp, _i32, _i64, _u32, _u64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_uint32, ctypes.c_uint64


def _fields(source, struct, skip=()):
    """Fields of a struct of the library's sources, in order."""
    src = open(os.path.join(ROOT, "paper_2606_17059_amd", "csrc", source)).read()
    body = re.search(r"struct %s \{(.*?)\n\};" % struct, src, flags=re.S).group(1)
    types = {"unsigned long long": _u64, "long long": _i64, "uint32_t": _u32}
    out = []
    for line in re.sub(r"//[^\n]*", "", body).split(";"):
        m = re.match(r"\s*(unsigned long long|long long|uint32_t)\s+(.+)", line, flags=re.S)
        if m:
            out += [(n.strip(), types[m.group(1)]) for n in m.group(2).split(",")]
    return out


def _struct(source, name):
    return type(name, (ctypes.Structure,), {"_fields_": _fields(source, name)})


Counters = _struct("merge_kernels.h", "MergeCounters")
Small = _struct("small_merge.h", "SmallStatus")
Walk = _struct("tree_walk.h", "WalkStatus")
Evict = _struct("tree_walk.h", "EvictStatus")
Compact = _struct("compact_kernels.h", "CompactState")


def build(out_dir):
    from paper_2606_17059_amd import build as B
    objs = [os.path.join(B.BUILD_DIR, n + ".o") for n in B.HIP_SOURCES + ["forest_host"]]
    if not all(map(os.path.exists, objs)):
        B.build()
    so = os.path.join(str(out_dir), "libhost_paths.so")
    cmd = ["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Wno-unused-result", "-D__HIP_PLATFORM_AMD__",
           "-isystem", os.path.join(ROCM, "include"), os.path.join(ROOT, "tests", "c", "host_runtime.cpp"), *objs,
           "-Wl,-Bsymbolic", "-Wl,-z,defs", "-o", so]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    return so


class HostRuntime:
    """L: the library with its entry points declared.  launches: kernel names since
    clear().  on[name] = f(args) plays the kernel whose name contains it; args are
    the addresses of its arguments (see arg, at)."""

    def __init__(self, so, monkeypatch):
        from paper_2606_17059_amd import router as R
        monkeypatch.setattr(R, "_lib_handle", None)
        monkeypatch.setattr(R, "LIB_PATH", so)
        self.R, self.L = R, R.lib()
        self.L.host_runtime_used.restype = self.L.host_runtime_refused.restype = ctypes.c_size_t
        self.L.host_runtime_limit.argtypes = [ctypes.c_size_t]
        self.launches = []
        self.errors = []
        self.on = {"stage_copy_kernel": self._stage, "set_used_kernel": self._set_used,
                   "small_merge_kernel": self.small_merge(), "compact_counters_kernel": self._compact_counters}
        hook = ctypes.CFUNCTYPE(None, ctypes.c_char_p, ctypes.POINTER(_vp), ctypes.c_uint, ctypes.c_uint)(self._hook)
        self._keep = hook
        self.L.host_runtime_hook(hook)
        self.limit(None)

    def _hook(self, name, args, grid, block):
        name = name.decode()
        self.launches.append(name)
        for k, f in self.on.items():
            if k in name:
                try:
                    f(args)
                except BaseException as e:  # not through the C caller
                    self.errors.append(repr(e))

    def clear(self):
        self.launches = []

    def launched(self, name):
        return sum(name in x for x in self.launches)

    def limit(self, bytes_):
        """Device memory there is (None: any amount)."""
        self.L.host_runtime_limit(ctypes.c_size_t(-1).value if bytes_ is None else bytes_)

    def used(self):
        return self.L.host_runtime_used()

    def refused(self):
        return self.L.host_runtime_refused()

    @staticmethod
    def arg(args, i, ctype=_vp):
        return ctypes.cast(args[i], ctypes.POINTER(ctype))[0]

    @classmethod
    def at(cls, args, i, struct):
        """The struct that pointer argument i points to."""
        return struct.from_address(cls.arg(args, i))

    def _stage(self, args):
        ctypes.memmove(self.arg(args, 1), self.arg(args, 0), 4 * self.arg(args, 2, _i32))

    def _set_used(self, args):
        c = self.at(args, 0, Counters)
        c.n_nodes, c.n_pool, c.overflow = self.arg(args, 1, _u64), self.arg(args, 2, _u64), 0

    def _compact_counters(self, args):
        c, S = self.at(args, 0, Counters), self.at(args, 1, Compact)
        c.n_nodes, c.n_pool = S.hi, S.n_pool

    def compacts_to(self, nodes, pool):
        """Compactions find that many live records and label tokens."""
        def play(index):
            def f(args):
                S = self.at(args, index, Compact)
                ctypes.memset(ctypes.addressof(S), 0, ctypes.sizeof(S))
                S.lo = S.hi = nodes
                S.n_pool = pool
            return f
        self.on["compact_small_kernel"] = play(5)
        self.on["compact_lab_scan_kernel"] = play(0)

    def walk_counts(self, tokens):
        """The one-launch walk finds a tree of that many tokens."""
        def play(args):
            w = Walk.from_address(self.arg(args, 5))
            w.done, w.tokens = 1, tokens
        self.on["tree_walk_kernel"] = play

    def walk_finds(self, nodes, leaves=0):
        """The level-by-level walk finds that many nodes and leaves at its first level;
        the one-launch walk and eviction report that the tree is too large for them."""
        def level(args):
            c = (_i32 * 3).from_address(self.arg(args, 9))
            c[0], c[1], c[2] = 0, leaves, nodes
        self.on["export_level_kernel"] = level
        self.on["tree_walk_kernel"] = lambda args: ctypes.memset(self.arg(args, 5), 0, ctypes.sizeof(Walk))
        self.on["evict_kernel"] = lambda args: ctypes.memset(self.arg(args, 7), 0, ctypes.sizeof(Evict))

    def evicts(self, tokens):
        """A player of the one-workgroup evictions, which evict that many tokens."""
        def play(args):
            c, out = self.at(args, 6, Counters), self.at(args, 7, Evict)
            out.done, out.evicted, out.n_nodes = 1, tokens, c.n_nodes
        return play

    def size_is(self, tokens):
        """Tree sizes that the pass over the records finds."""
        def size(args):
            _u64.from_address(self.arg(args, 4)).value = tokens
        self.on["tree_size_kernel"] = size

    def small_merge(self, *replies, **fields):
        """A player of the one-workgroup merge: every launch reports `fields` (by
        default that all is done in one round), the first ones with the given replies
        on top; add_nodes and add_pool advance the counters."""
        todo = list(replies)

        def play(args):
            f = {"done": 1, "rounds": 1, **fields, **(todo.pop(0) if todo else {})}
            c, out = self.at(args, 3, Counters), self.at(args, 7, Small)
            nodes, pool = c.n_nodes + f.pop("add_nodes", 0), c.n_pool + f.pop("add_pool", 0)
            ctypes.memset(ctypes.addressof(c), 0, ctypes.sizeof(c))
            ctypes.memset(ctypes.addressof(out), 0, ctypes.sizeof(out))
            c.n_nodes = out.n_nodes = nodes
            c.n_pool = out.n_pool = pool
            for k, v in f.items():
                setattr(out, k, v)
        return play

    def forest(self, peers, snapshots=()):
        f = Forest(self, peers)
        for p, seqs in enumerate(snapshots):
            f.load(p, seqs)
        return f

    def large_merge(self, f, nodes, pool):
        """A merge of 65 sequences that adds that many records and label tokens: the
        forest grows to them (a refused request, a walk's tally), then uses them."""
        tallies = [(1, pool), (0, 0)]

        def tally(args):
            c = self.at(args, 2, Counters)
            c.n_split, c.pool_need = tallies.pop(0) if tallies else (0, 0)
        self.on["merge_tally_kernel"] = tally
        self.on["small_merge_kernel"] = self.small_merge(dict(done=0, overflow=1, add_nodes=nodes))
        assert f.merge(65) == 0
        i = f.info()
        self.on["small_merge_kernel"] = self.small_merge(dict(add_nodes=nodes - i.num_nodes, add_pool=pool))
        assert f.merge(65) == 0
        assert f.info().num_nodes == nodes


class Forest:
    """Entry points on host arrays; every call returns its status."""

    def __init__(self, rt, peers):
        self.rt, self.L = rt, rt.L
        h = _vp()
        assert self.L.pr_forest_create(peers, ctypes.byref(h)) == 0
        self.h = h

    def close(self):
        self.L.pr_forest_destroy(self.h)
        assert not self.rt.errors, self.rt.errors

    def error(self):
        return self.L.pr_last_error().decode()

    def info(self):
        i = self.rt.R.ForestInfo()
        assert self.L.pr_forest_info_get(self.h, ctypes.byref(i)) == 0
        return i

    @staticmethod
    def csr(seqs):
        off = np.zeros(len(seqs) + 1, np.int64)
        np.cumsum([len(s) for s in seqs], out=off[1:])
        return np.concatenate([np.asarray(s, np.int32) for s in seqs] or [np.zeros(0, np.int32)]), off

    def load(self, p, seqs):
        t, o = self.csr(seqs)
        return self.L.pr_load_snapshot(self.h, p, t.ctypes.data if t.size else None, o.ctypes.data, len(seqs))

    def merge(self, n, tokens=1, peer=0):
        """n inserts of `tokens` tokens each."""
        pe = np.full(n, peer, np.int32)
        t, o = np.zeros(max(n * tokens, 1), np.int32), np.arange(n + 1, dtype=np.int64) * tokens
        return self.L.pr_merge(self.h, pe.ctypes.data, t.ctypes.data, n * tokens, o.ctypes.data, n, None)

    def load_device(self, p, n, tokens=1):
        """A snapshot of n sequences that is on the device."""
        t, o = np.zeros(max(n * tokens, 1), np.int32), np.arange(n + 1, dtype=np.int64) * tokens
        return self.L.pr_load_snapshot_device(self.h, p, t.ctypes.data, n * tokens, o.ctypes.data, n, None)

    def touch(self, n, tokens=1):
        t, o = np.zeros(max(n * tokens, 1), np.int32), np.arange(n + 1, dtype=np.int64) * tokens
        return self.L.pr_touch(self.h, t.ctypes.data, n * tokens, o.ctypes.data, n, None)

    def evict(self, n):
        e = _i64(-1)
        return self.L.pr_evict_lru(self.h, n, ctypes.byref(e), None), e.value

    def tokens(self, p):
        v = _i64(-1)
        return self.L.pr_tree_tokens(self.h, p, ctypes.byref(v), None), v.value

    def compact(self):
        return self.L.pr_forest_compact(self.h, None, None, None)

    def export(self, p, seqs_cap=None, tokens_cap=0):
        """Sizes alone, or (with seqs_cap) into buffers of those capacities."""
        s, t = _i64(-1), _i64(-1)
        if seqs_cap is None:
            st = self.L.pr_export_snapshot(self.h, p, None, 0, None, 0, ctypes.byref(s), ctypes.byref(t), None)
        else:
            tok, off = np.zeros(max(tokens_cap, 1), np.int32), np.zeros(max(seqs_cap, 1), np.int64)
            st = self.L.pr_export_snapshot(self.h, p, tok.ctypes.data, tokens_cap, off.ctypes.data, seqs_cap,
                                           ctypes.byref(s), ctypes.byref(t), None)
        return st, s.value, t.value
