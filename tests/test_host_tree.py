"""Host logic of a tree's life, on a stand-in for the GPU runtime
(host_runtime.cpp: no GPU, launches do nothing): what a failed rebuild leaves
behind.  Each test body runs in a process of its own, which loads the
stand-in before the library."""
import os
import subprocess
import sys

import pytest

from conftest import ROOT

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes, sys
rt = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
rt.rt_calls.restype = ctypes.c_char_p
libc = ctypes.CDLL(None)
libc.malloc.restype, libc.malloc.argtypes, libc.free.argtypes = ctypes.c_void_p, [ctypes.c_size_t], [ctypes.c_void_p]
import paper_1106_2176_amd as fmm
L = fmm.lib()
P = ctypes.c_void_p(16)     # a pointer that nothing here reads
A, B = ctypes.c_void_p(32), ctypes.c_void_p(64)  # streams

def counts(adaptive, n, nbox=0, lev=0):
    # what a build reads: two counters; adaptive, from the fifth word on: the
    # first box of each level, boxes, boxes + leaves, bad positions, then the
    # lengths of three lists and the split boxes of each level
    def words(w):
        rt.rt_counts((ctypes.c_uint32 * 132)(*w), 132)
    if not adaptive:
        return words([0, 1])
    first = [(8 ** l - 1) // 7 for l in range(lev + 1)] + [nbox] * (10 - lev)
    words([0] * 4 + first + [nbox, 2 * nbox - 1, 0])
    words([0] * 4 + [9 * nbox, nbox, nbox] + [8 ** l for l in range(lev)] + [0] * (1 + 8 * (lev - 1)))

def build(cfg, n, h, stream=A):
    return L.fmm_build_tree(ctypes.byref(cfg), n, fmm.FMM_F64, P, stream, ctypes.byref(h))
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rt") / "host_runtime.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-w", "-o", so, os.path.join(HERE, "host_runtime.cpp")], check=True)
    return so


def _run(runtime, body, *args):
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, runtime, *map(str, args)], cwd=ROOT, timeout=100,
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("adaptive,failing", [(False, 0), (False, 1), (True, 0), (True, 1), (True, 2)])
def test_a_tree_whose_rebuild_failed_is_refused_until_one_succeeds(runtime, adaptive, graph, failing):
    """The failing-th allocation of a rebuild for more particles finds no
    memory: every call that would read the tree's buffers is refused before
    any launch, and a rebuild that succeeds makes the tree usable again."""
    _run(runtime, """
adaptive, graph, failing = (int(x) for x in sys.argv[2:])
left = [1 << 30]
def alloc(nbytes, stream, ctx):
    left[0] -= 1
    return libc.malloc(nbytes) if left[0] >= 0 else None
def free(ptr, stream, ctx):
    libc.free(ptr)
cbs = (fmm.ALLOC_FN(alloc), fmm.FREE_FN(free))
cfg = fmm.make_config(p=4, leaf_max=8, precision="fp64", adaptive=bool(adaptive), graph=bool(graph), allocator=cbs)
h = ctypes.c_void_p()
def calls():
    i, s = fmm.TreeInfo(), (ctypes.c_int64 * 6)()
    w = (ctypes.c_uint32 * 4_000_000)()
    out = [L.fmm_evaluate(h, P, P, P, fmm.VEC_FIELD, A), L.fmm_evaluate_noalloc(h, P, P, P, fmm.VEC_FIELD, A),
           L.fmm_backward(h, P, P, P, P, P, A), L.fmm_tree_info(h, ctypes.byref(i)), L.fmm_tree_export(h, w, w)]
    return out + [L.fmm_tree_export_adaptive(h, s, None, None, None, None)] if adaptive else out
counts(adaptive, 3000, 585, 3)
assert build(cfg, 3000, h) == fmm.FMM_OK
assert not any(calls())
left[0] = failing
counts(adaptive, 50_000, 37449, 5)
rc = build(cfg, 50_000, h)
assert rc == fmm.FMM_ENOMEM and h.value
before = rt.rt_launches()
left[0] = 1 << 30
got = calls()
assert all(r == fmm.FMM_EDEVICE for r in got), got
assert rt.rt_launches() == before
rt.rt_forget_counts()
counts(adaptive, 3000, 585, 3)
assert build(cfg, 3000, h) == fmm.FMM_OK
assert not any(calls())
L.fmm_tree_destroy(h)
""", int(adaptive), int(graph), failing)


@pytest.mark.parametrize("adaptive", [False, True])
@pytest.mark.parametrize("other", [False, True])
def test_destroy_waits_for_the_trees_device(runtime, adaptive, other):
    """A tree that another stream has used is destroyed while another device
    is current: its own device is waited for, once, and the caller's stays
    current.  A tree used on its build's stream alone is not waited for."""
    _run(runtime, """
adaptive, other = (int(x) for x in sys.argv[2:])
h = ctypes.c_void_p()
cfg = fmm.make_config(p=4, leaf_max=8, precision="fp64", adaptive=bool(adaptive), allocator="library")
counts(adaptive, 3000, 585, 3)
rt.hipSetDevice(2)
assert build(cfg, 3000, h) == fmm.FMM_OK
assert L.fmm_evaluate(h, P, P, P, fmm.VEC_FIELD, B if other else A) == fmm.FMM_OK
rt.hipSetDevice(1)
seen = len(rt.rt_calls())
L.fmm_tree_destroy(h)
calls = rt.rt_calls()[seen:].decode().split()
assert [c for c in calls if c.startswith("wait")] == (["wait2"] if other else []), calls
d = ctypes.c_int()
rt.hipGetDevice(ctypes.byref(d))
assert d.value == 1
""", int(adaptive), int(other))


def test_destroy_allocates_nothing(runtime):
    """Destroying trees needs no host memory (nothing may be thrown out of
    the C interface); words and events are handed on to at most eight later
    trees, the others' given back."""
    _run(runtime, """
cfg = fmm.make_config(p=4, leaf_max=8, precision="fp64", allocator="library")
trees = [ctypes.c_void_p() for _ in range(10)]
for h in trees:
    counts(False, 3000)
    assert build(cfg, 3000, h) == fmm.FMM_OK
rt.rt_no_memory(1)
for h in trees:
    L.fmm_tree_destroy(h)
rt.rt_no_memory(0)
assert rt.rt_calls().count(b"unpin") == 2
""")
