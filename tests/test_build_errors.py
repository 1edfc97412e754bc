"""What an error leaves behind, with a stand-in for the HIP runtime (fake_hip.cpp) in a process of its own: no GPU takes part."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

_BEGIN = """
import ctypes, sys
sys.path.insert(0, sys.argv[2])
fake = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)   # found before the runtime that the library names
import numpy as np
from paper_1904_03329_amd import binding as B
fake.fake_pending.restype = fake.fake_into.restype = ctypes.c_long
def start(copy=0, wait=0):
    fake.fake_start(ctypes.c_long(copy), ctypes.c_long(wait))
def memory(n):
    a = np.zeros(n + 256, dtype=np.uint8)
    return a[-a.ctypes.data % 256:][:n]
def code(call):
    try:
        call()
    except B.HbcsfError as e:
        return e.code
    return 0
dims, nnz = (50, 40, 30), 3000
rng = np.random.default_rng(1)
inds = [x.astype(np.uint32) for x in np.unravel_index(rng.choice(60000, nnz, replace=False), dims)]
vals = rng.uniform(-1, 1, nnz).astype(np.float32)
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-o", so,
                           os.path.join(HERE, "fake_hip.cpp")])

    def call(script):
        r = subprocess.run([sys.executable, "-c", _BEGIN + script, so, os.path.dirname(HERE)], capture_output=True, text=True,
                           timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr

    return call


def test_nothing_is_enqueued_after_a_device_build_has_failed(run):
    """Memory is refused for the modes and for the words of state (the kernels of the modes before are enqueued by then), an
    allocation raises, the arena is too small, and every copy and wait of a build fails once: the memory is the caller's again,
    so all that was enqueued must have been waited for."""
    run("""
arena, workspace = B.device_build_bytes(dims, nnz)
ws = memory(workspace)
def build(allocate):
    return B.build_format_device_pieces(dims, nnz, [x.ctypes.data for x in inds], vals.ctypes.data, allocate, ws.ctypes.data,
                                        workspace)
pieces = []
def give(n):
    pieces.append(memory(n))
    return pieces[-1].ctypes.data
start()
h = build(give)
assert fake.fake_pending() == 0 and len(pieces) == 4   # three modes, the words of state
B.lib().hbcsf_free(h)
for refused in range(4):
    left = [refused]
    def some(n):
        left[0] -= 1
        return give(n) if left[0] >= 0 else None
    start()
    assert code(lambda: build(some)) == -3
    assert fake.fake_pending() == 0, refused
start()
assert code(lambda: build(lambda n: give(n) + 128)) == -1
assert fake.fake_pending() == 0
def raises(n):
    raise MemoryError
start()
try:
    build(raises)
    assert False
except MemoryError:
    pass
assert fake.fake_pending() == 0
need = sum(p.size for p in pieces[:4])
for less in (256, need // 2):
    small = memory(need)
    start()
    assert code(lambda: B.build_format_device(dims, nnz, [x.ctypes.data for x in inds], vals.ctypes.data, small.ctypes.data,
                                              need - less, ws.ctypes.data, workspace)) == -3
    assert fake.fake_pending() == 0
for opts in ({}, dict(hybrid_granularity=1)):
    arena, workspace = B.device_build_bytes(dims, nnz, **opts)
    ws = memory(workspace)
    for what in ("copy", "wait"):
        for nth in range(1, 30):
            start(**{what: nth})
            c = code(lambda: B.build_format_device_pieces(dims, nnz, [x.ctypes.data for x in inds], vals.ctypes.data, give,
                                                          ws.ctypes.data, workspace, **opts))
            assert fake.fake_pending() == 0, (opts, what, nth)
            if c == 0:
                break
            assert c == -5
        assert nth > 3
""")


def test_a_failed_upload_or_move_leaves_the_handle_where_it_was(run):
    """Every copy and wait of a second upload and of a move fails once.  The handle then still reads the arena it had: a further
    move copies that arena's arrays, and an MTTKRP launch is given pointers into it, of the words of state too, and none into the
    memory of the call that failed."""
    run("""
h = B.build_format(dims, inds, vals)
n = B.device_bytes(h)
start()
first = memory(n)
B.upload(h, first.ctypes.data, n)
arrays = first.copy()
facs = [rng.uniform(size=(d, 32)).astype(np.float32) for d in dims]
out = memory(4 * 32 * max(dims))
def pointers(arena):
    fake.fake_range(ctypes.c_void_p(arena.ctypes.data), ctypes.c_void_p(arena.ctypes.data + n))
    B.mttkrp(h, 0, 32, [f.ctypes.data for f in facs], out.ctypes.data)
    into = fake.fake_into()
    fake.fake_range(None, None)
    return into
uses = pointers(first)
assert uses > 10
held = first
for call in (B.upload, B.relocate):
    for what in ("copy", "wait"):
        for nth in range(1, 9):
            other = memory(n)
            start(**{what: nth})
            c = code(lambda: call(h, other.ctypes.data, n))
            assert fake.fake_pending() == 0
            start()
            if c == 0:
                assert pointers(other) == uses and pointers(held) == 0
                held = other
                break
            assert c == -5
            assert pointers(held) == uses and pointers(other) == 0, (call, what, nth)
            other[:] = 0xff
            moved = memory(n)
            B.relocate(h, moved.ctypes.data, n)
            assert np.array_equal(moved, arrays), (call, what, nth)
            held = moved
        assert nth > 1
""")


def test_workspace_of_blocked_builds(run):
    """Blocked orders of 64-bit keys are sorted in the pair sort's own buffers: no workspace for a fourth pair of 12 bytes a nonzero,
    which only the per-fiber choice uses."""
    run("""
long, nnz = (12_000_000, 9_000_000, 100), 10_000_000   # as many slices as nonzeros, blocked or not
def workspace(**opts):
    return B.device_build_bytes(long, nnz, **opts)[1]
start()
assert workspace(mid_blocking=4) == workspace()
both = workspace(mid_blocking=4, hybrid_granularity=1)
assert both == workspace(hybrid_granularity=1) and both > workspace() + 12 * nnz
""")
