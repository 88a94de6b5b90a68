"""The cache of long work lists on the CPU: the library's host code linked with
a stand-in for the GPU (stub_runtime.cpp) whose stream runs when the test says
so and whose launches check every range that the kernels write."""

import ctypes
import os
import shutil
import subprocess
import threading
import time

import numpy as np
import pytest

import paper_2512_20968_amd as ma
from paper_2512_20968_amd import _binding

from helpers import concurrency_tiles, device_list_tiles, plan_cache_tiles

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests")


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = tmp_path_factory.mktemp("host") / "libhost.so"
    csrc = os.path.join(ROOT, "paper_2512_20968_amd", "csrc")
    subprocess.run(
        [gxx, "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC",
         "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-I",
         csrc, "-I", "/opt/rocm/include", os.path.join(csrc, "host.cpp"),
         os.path.join(HERE, "stub_runtime.cpp"), "-o", str(out),
         "-Wl,-Bsymbolic"], check=True)
    return out


class Host:
    """One copy of the library, with a cache of its own."""

    FAKE = [ctypes.c_void_p(0x10000 * (i + 1)) for i in range(10)]

    def __init__(self, path):
        lib = ctypes.CDLL(str(path))
        for name in ("tile_fwd", "tile_bwd", "chunk_fwd", "chunk_bwd",
                     "fwd_workspace_size", "bwd_workspace_size",
                     "chunk_fwd_workspace_size", "chunk_bwd_workspace_size",
                     "tile_fwd_noalloc", "last_error"):
            fn = getattr(lib, "mesh_attn_" + name)
            fn.restype, fn.argtypes = _binding._SIGNATURES["mesh_attn_" + name]
        lib.stub_workspace.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
        lib.stub_run.argtypes = [ctypes.c_void_p]
        self.lib = lib
        self.bufs = [np.empty(0, np.uint8)]  # pending copies may use old ones

    def workspace(self, nbytes):
        if self.bufs[-1].size < nbytes + 256:
            self.bufs.append(np.empty(nbytes + 256, np.uint8))
        at = (self.bufs[-1].ctypes.data + 255) // 256 * 256
        self.lib.stub_workspace(at, nbytes)
        return at

    @staticmethod
    def _list(idx):
        return [(ctypes.c_int32 * len(idx))(*idx), len(idx)]

    def call(self, pass_, prob, q_idx, kv_idx, ws_bytes=None, chunk=None,
             stream=None, check=True):
        """Runs a forward (0) or backward (1); returns the status."""
        pr = ma.Problem.make(prob)
        q, nq = self._list(q_idx)
        kv, nkv = self._list(kv_idx)
        kind = "chunk_" if chunk else ""
        name = kind + ("bwd" if pass_ else "fwd")
        if ws_bytes is None:
            ws_bytes = getattr(self.lib, f"mesh_attn_{name}_workspace_size")(
                ctypes.byref(pr), nq, nkv)
        ws = self.workspace(ws_bytes)
        head = [ctypes.byref(pr), q, nq, kv, nkv]
        f = self.FAKE
        if chunk:
            head.append(ctypes.byref(_binding.Chunk(*chunk)))
        if pass_:
            args = f[:9] + [0, ws, ws_bytes, stream]
        elif chunk:
            args = f[:5] + [0, ws, ws_bytes, stream]
        else:
            args = f[:4] + [0, f[4], ws, ws_bytes, stream]
        fn = getattr(self.lib,
                     "mesh_attn_" + (name if chunk else "tile_" + name))
        st = fn(*head, *args)
        if check:
            assert st == 0, self.lib.mesh_attn_last_error()
        return st

    def call_noalloc(self, prob, q_idx, kv_idx):
        pr = ma.Problem.make(prob)
        f = self.FAKE
        return self.lib.mesh_attn_tile_fwd_noalloc(
            ctypes.byref(pr), *self._list(q_idx), *self._list(kv_idx), *f[:4],
            0, f[4], None)

    def last(self):
        out = (ctypes.c_int32 * 14)()
        self.lib.stub_last(out)
        return tuple(out[:7]), tuple(out[7:])

    def counts(self):
        out = (ctypes.c_int32 * 4)()
        self.lib.stub_counts(out)
        return dict(zip(("out_of_range", "stale", "pinned", "launches"), out))

    def run(self, *streams):
        for s in streams:
            self.lib.stub_run(s)


@pytest.fixture
def host(library, tmp_path):
    # A copy per test: its own globals, so an empty cache.
    return Host(shutil.copy(library, tmp_path / "libhost.so"))


@pytest.fixture
def other(library, tmp_path):
    return Host(shutil.copy(library, tmp_path / "libother.so"))


def _prob(n, P, hq, hkv, d, causal=0, layout=0):
    return dict(num_partitions=n, partition_len=P, num_q_heads=hq,
                num_kv_heads=hkv, head_dim=d, causal=causal, layout=layout,
                softmax_scale=0.125)


# Lists too long for the kernel arguments, of few items, long enough to be
# split; the numbers of pieces and partials of the two head dims differ.
SPLIT_LONG = [
    (0, _prob(8, 4096, 4, 4, 64), [0, 1, 2, 3, 4], [0, 1]),
    (0, _prob(64, 1024, 2, 1, 64, 1, 1), list(range(63, 23, -1)),
     list(range(0, 60, 5))),
    (1, _prob(8, 4096, 2, 2, 64), [0, 1, 2, 3], [0, 1]),
    (1, _prob(8, 2048, 8, 2, 64, 1), [3, 1, 5], [2, 3, 0, 1]),
]


@pytest.mark.parametrize("first", [64, 128])
@pytest.mark.parametrize("pass_,prob,q,kv", SPLIT_LONG)
def test_tiles_that_differ_in_head_dim_have_plans_of_their_own(
        host, other, pass_, prob, q, kv, first):
    second = 192 - first
    host.call(pass_, dict(prob, head_dim=first), q, kv)
    assert not any(o[0] for o in host.last())  # not in the kernel arguments
    assert any(o[5] > 0 for o in host.last())  # split
    host.call(pass_, dict(prob, head_dim=second), q, kv)
    other.call(pass_, dict(prob, head_dim=second), q, kv)
    # What the second head dim gets does not depend on the first call.
    assert host.last() == other.last()
    assert host.counts()["out_of_range"] == 0


# A tile whose list is too long for the kernel arguments: 128 Q blocks.
LONG = _prob(2048, 256, 1, 1, 64)


def _long_tile(i):
    return LONG, list(range(128)), [i]


def test_evicted_lists_keep_their_buffers_until_they_have_been_read(host):
    """More tiles than the cache holds, on two streams: no buffer is handed out
    again while a copy from it is pending, and all are once none is."""
    for i in range(1100):
        host.call(i % 2, *_long_tile(i), stream=1 + i % 3 // 2)
    assert host.counts()["pinned"] == 1100  # none could be recycled
    # Stream 1 goes on: of the 76 lists evicted so far (the first ones), those
    # that it has read give their buffers to the next tiles of their pass.
    host.run(1)
    for i in range(1100, 1140):
        host.call(i % 2, *_long_tile(i), stream=1)
    assert host.counts()["pinned"] == 1100
    for i in range(1140, 1400):
        host.call(i % 2, *_long_tile(i), stream=1)
        host.run(1)
    before = host.counts()["pinned"]
    assert before < 1250
    host.run(2)
    for i in range(1400, 2000):
        host.call(i % 2, *_long_tile(i), stream=1 + i % 2)
        host.run(1, 2)
    assert host.counts() == dict(out_of_range=0, stale=0, pinned=before,
                                 launches=2000)


def test_a_list_seen_again_is_the_same(host, other):
    host.call(0, *_long_tile(0))
    first = host.last()
    for i in range(1, 1100):
        host.call(0, *_long_tile(i))
        host.run(None)
    pinned = host.counts()["pinned"]
    host.call(0, *_long_tile(0))  # evicted since, built again
    assert host.last() == first and host.counts()["pinned"] == pinned
    host.call(0, *_long_tile(0))
    host.run(None)
    assert host.last() == first and host.counts()["stale"] == 0


def test_the_gpu_tests_of_the_cache_use_it(host):
    cfg, kv_lists = plan_cache_tiles()
    assert len({tuple(kv) for kv in kv_lists}) == 1100
    for pass_ in (0, 1):
        for kv in kv_lists[::50]:
            host.call(pass_, cfg.problem(), cfg.q_idx, kv)
            assert not any(o[0] for o in host.last())
    used = {}
    for i, c in enumerate(concurrency_tiles()):
        for pass_ in (0, 1):
            pinned = host.counts()["pinned"]
            host.call(pass_, c.problem(), c.q_idx, c.kv_idx)
            used[i, pass_] = host.counts()["pinned"] > pinned
    assert all(used[i, 0] == (i % 2 == 1) for i in range(8))
    assert all(used[i, 1] for i in (0, 1, 4, 5))


def test_a_launch_does_not_hold_up_other_threads(host):
    """While one call is inside its launch (a full queue may hold it there),
    another thread's call with a long list gets through."""
    host.workspace(1 << 20)
    done = []

    def other_call():
        host.call(0, *_long_tile(1), ws_bytes=1 << 20, stream=2)
        done.append(True)

    @ctypes.CFUNCTYPE(None)
    def inside_the_launch():
        th = threading.Thread(target=other_call, daemon=True)
        th.start()
        th.join(20)

    host.lib.stub_hook(inside_the_launch)
    host.call(0, *_long_tile(0), ws_bytes=1 << 20, stream=1)
    assert done == [True]
    host.run(1, 2)
    assert host.counts() == dict(out_of_range=0, stale=0, pinned=2, launches=2)


@pytest.mark.parametrize("pass_", [0, 1])
def test_a_failed_event_after_the_launch_is_not_a_failed_call(host, pass_):
    host.lib.stub_fail(0, 1)
    host.call(pass_, *_long_tile(0), stream=1)
    assert host.counts()["launches"] == 1
    # Nothing says when that call has read its list, so it keeps its buffer,
    # also after the list has been evicted.
    for i in range(1, 1100):
        host.call(pass_, *_long_tile(i), stream=2)
        host.run(2)
    host.run(1)
    assert host.counts()["stale"] == 0


def test_a_failed_launch_is_reported(host):
    host.lib.stub_fail(1, 0)
    assert host.call(0, *_long_tile(0), check=False) == _binding.MA_ERR_HIP
    assert b"launch" in host.lib.mesh_attn_last_error()
    host.call(0, *_long_tile(0))
    host.run(None)
    assert host.counts()["stale"] == 0


# Heads, head dim, and the partitions of a large and of a small tile: the large
# one has too many items to split any.
SMALLER = [(4, 1, 128, (40, 16), (1, 16)), (8, 8, 64, (20, 20), (2, 20)),
           (5, 5, 128, (40, 8), (2, 8))]


@pytest.mark.parametrize("pass_", [0, 1])
@pytest.mark.parametrize("hq,hkv,d,large,small", SMALLER)
def test_a_workspace_serves_every_smaller_tile(host, other, pass_, hq, hkv, d,
                                               large, small):
    """A workspace sized for a tile is as good for one of fewer partitions, and
    for every chunk task of either, as one of its own."""
    prob = _prob(40, 4096, hq, hkv, d)
    size = getattr(ma, f"mesh_attn_{'bwd' if pass_ else 'fwd'}_workspace_size")
    need = size(prob, *large)
    assert need >= size(prob, *small)
    q, kv = list(range(small[0])), list(range(20, 20 + small[1]))
    for chunk in (None, (0, 1, 1, 2), (1, 2, 0, 4)):
        host.call(pass_, prob, q, kv, ws_bytes=need, chunk=chunk)
        other.call(pass_, prob, q, kv, chunk=chunk)
        assert host.last() == other.last()
        if chunk is None:
            assert any(o[5] > 0 for o in host.last())  # split
    assert host.counts()["out_of_range"] == 0


def test_workspace_sizes_grow_with_the_tile():
    for name in ("fwd", "bwd", "chunk_fwd", "chunk_bwd"):
        size = getattr(ma, f"mesh_attn_{name}_workspace_size")
        for P, hq, hkv, d in ((256, 21, 7, 64), (1024, 1, 1, 128),
                              (4096, 32, 8, 128), (4096, 64, 64, 64)):
            prob = _prob(64, P, hq, hkv, d)
            got = np.array([[size(prob, nq, nkv) for nkv in range(1, 40)]
                            for nq in range(1, 40)])
            assert (np.diff(got, axis=0) >= 0).all()
            assert (np.diff(got, axis=1) >= 0).all()


def test_a_cached_list_is_not_built_again(host):
    """A call whose list is in the cache finds it there without building it
    (choosing the cut of this tile takes tens of microseconds), so it takes
    about as long as the smallest call: the fastest of many, by the clock of
    this process's CPU time."""
    tiny = (0, _prob(4, 256, 4, 4, 64), [0, 1], [0, 1])
    long = (0, _prob(64, 4096, 1, 1, 128, 1), list(range(50, 55)),
            list(range(40)))

    def fastest(args):
        host.call(*args)  # builds the list
        best = float("inf")
        for _ in range(400):
            t = time.process_time_ns()
            host.call(*args, ws_bytes=1 << 28)
            best = min(best, time.process_time_ns() - t)
            host.run(None)
        return best

    # 40 more indexes to pass, a lookup, a copy and an event.
    assert fastest(long) < 2.5 * fastest(tiny)


@pytest.mark.parametrize("nq,nkv,P,heads,split", [
    (3, 1, 4096, 4, False), (4, 1, 4096, 4, False), (3, 1, 2048, 8, False),
    (3, 2, 4096, 4, False), (3, 4, 1024, 14, True), (2, 2, 2048, 8, True),
    (2, 2, 1024, 14, True), (4, 4, 4096, 4, True)])
def test_items_with_a_compute_unit_each(host, nq, nkv, P, heads, split):
    """Head dim 64, at most 256 items: they are cut where that measured faster
    than leaving them whole."""
    host.call(0, _prob(8, P, heads, heads, 64), list(range(nq)),
              list(range(nkv)))
    assert (host.last()[0][5] > 0) == split


@pytest.mark.parametrize("nq,nkv,P,hq,hkv,split", [
    (3, 8, 4096, 4, 1, True), (3, 2, 2048, 8, 8, True),
    (3, 4, 4096, 14, 2, True), (4, 4, 4096, 8, 8, False),
    (1, 4, 4096, 16, 16, False)])
def test_dq_items_beside_dkdv_items(host, nq, nkv, P, hq, hkv, split):
    """Head dim 128, equal items, dK/dV items whole: dQ items that fill whole
    rounds of their places stay whole, others are cut."""
    host.call(1, _prob(8, P, hq, hkv, 128), list(range(nq)), list(range(nkv)))
    dq, dkdv = host.last()
    assert dkdv[5] == 0 and (dq[5] > 0) == split


def test_noalloc_limit_is_the_headers_formula(host):
    """The allocation-free forward serves the tiles within its documented limit
    and no other, and their lists lie inside the scratch array."""
    def up(x):
        return (x + 255) // 256 * 256

    def fits(P, hq, nq, nkv):
        blocks = nq * P // 256
        return (blocks <= 4096 and
                up(4 * (blocks + 1)) + up(32 * blocks * nkv) +
                up(8 * (blocks * hq + 8)) + 256 <= 8 << 20)

    served = 0
    for P, hq, d in ((256, 1, 64), (4096, 32, 128), (1024, 7, 64),
                     (2048, 64, 128), (1024, 1, 64)):
        for nq in (1, 100, 128, 200, 255, 256):
            for nkv in (1, 30, 31, 62, 63, 64, 128, 255, 256):
                st = host.call_noalloc(_prob(512, P, hq, 1, d, 1), range(nq),
                                       range(nkv))
                ok = fits(P, hq, nq, nkv)
                served += ok
                assert st == (0 if ok else _binding.MA_ERR_UNSUPPORTED)
                assert ok or b"scratch" in host.lib.mesh_attn_last_error()
    assert 100 < served < 250
    assert host.counts()["out_of_range"] == 0


def _random_call(rng):
    P = 256 * int(rng.choice([1, 2, 3, 4, 5, 8, 12, 16, 32]))
    n = int(rng.integers(1, 40))
    nq, nkv = (int(min(n, rng.integers(1, 18))) for _ in range(2))
    hkv, g = int(rng.choice([1, 2, 3, 4, 7, 8, 16])), int(rng.choice([1, 2, 3, 8]))
    prob = _prob(n, P, hkv * g, hkv, int(rng.choice([64, 128])),
                 int(rng.integers(2)), int(rng.integers(2)))
    q, kv = ([int(x) for x in rng.permutation(n)[:k]] for k in (nq, nkv))
    chunk = None
    if rng.random() < 0.3:
        kq = int(rng.choice([x for x in (1, 2, 3, 4) if P % (256 * x) == 0]))
        kk = int(rng.choice([x for x in (1, 2, 4, 6) if P % (128 * x) == 0]))
        chunk = (int(rng.integers(kq)), kq, int(rng.integers(kk)), kk)
    return prob, q, kv, chunk


def test_the_gpu_test_of_device_built_lists_covers_the_slot_orders(host):
    modes = set()
    for c in device_list_tiles():
        assert host.call_noalloc(c.problem(), c.q_idx, c.kv_idx) == 0
        inline, _, _, mode, parts, splits, _ = host.last()[0]
        assert not inline and parts > 0 and splits > 0
        modes.add((mode, c.head_dim))
    assert {(0, 128), (1, 64), (2, 64), (2, 128)} <= modes
    assert c.nq * c.partition_len // 256 > 1024


def test_random_calls_stay_inside_their_workspace(host):
    """Forward, backward, chunk tasks and the allocation-free forward of random
    tiles, in workspaces of their own size, sized for a larger tile, and without
    room for all partial results: every range that a launch writes lies inside,
    and the allocation-free forward cuts as a workspace of full size does."""
    rng = np.random.default_rng(17)
    split = 0
    for _ in range(400):
        prob, q, kv, chunk = _random_call(rng)
        for pass_ in (0, 1):
            size = getattr(ma, f"mesh_attn_{'bwd' if pass_ else 'fwd'}"
                           "_workspace_size")
            own = size(prob, len(q), len(kv))
            for ws in (own, size(prob, len(q) + 3, len(kv) + 2),
                       int(own * rng.random())):
                st = host.call(pass_, prob, q, kv, ws_bytes=ws, chunk=chunk,
                               check=False)
                small = _binding.MA_ERR_WORKSPACE_TOO_SMALL
                assert st == 0 or (st == small and ws < own), (prob, q, kv, ws)
                host.run(None)
            if pass_ == 0 and chunk is None:
                host.call(0, prob, q, kv)
                want = host.last()[0][1:]  # inline or not
                host.run(None)
                if host.call_noalloc(prob, q, kv) == 0:
                    assert host.last()[0][1:] == want, (prob, q, kv)
                split += want[4] > 0
        assert host.counts()["out_of_range"] == 0, (prob, q, kv, chunk)
        assert host.counts()["stale"] == 0
    assert split > 40
