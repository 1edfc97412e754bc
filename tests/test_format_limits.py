"""What the host builder refuses, what it reports and what it holds (no GPU)."""
import os
import subprocess
import sys
import time

import numpy as np
import pytest

import format_walk as FW
from paper_1904_03329_amd import binding as B


def _corners(dims, nnz, seed):
    rng = np.random.default_rng(seed)
    inds = [rng.integers(0, d, size=nnz, dtype=np.uint64).astype(np.uint32) for d in dims]
    return inds, rng.uniform(-1, 1, nnz).astype(np.float32)


@pytest.mark.parametrize("bits, opts, built", [
    ((26, 26, 26, 26, 24), dict(), True),                       # 128 bits: the widest key
    ((26, 26, 26, 26, 25), dict(), False),
    ((30, 30, 30, 30, 30), dict(), False),
    ((26, 26, 26, 26, 22), dict(mid_blocking=2), True),          # 126 bits and a blocked mode's block number of 2
    ((26, 26, 26, 26, 22), dict(mid_blocking=3), False),
])
def test_keys_above_128_bits_are_refused(bits, opts, built):
    dims = tuple(1 << b for b in bits)
    inds, vals = _corners(dims, 300, 5)
    if not built:
        with pytest.raises(B.HbcsfError) as e:
            B.build_format(dims, inds, vals, **opts)
        assert e.value.code == -2
        return
    h = B.build_format(dims, inds, vals, **opts)
    try:
        for mode in range(len(dims)):
            fmt = FW.read_mode(h, mode, len(dims))
            cols, v = FW.expand_to_coo(fmt)
            got = np.stack([cols[fmt["level_mode"].index(m)].astype(np.int64) for m in range(len(dims))]
                           + [v.view(np.uint32).astype(np.int64)])
            want = np.stack([x.astype(np.int64) for x in inds] + [vals.view(np.uint32).astype(np.int64)])
            assert np.array_equal(got[:, np.lexsort(got[::-1])], want[:, np.lexsort(want[::-1])])
    finally:
        B.free(h)


def test_build_seconds_account_for_the_whole_call():
    """The modes' times add up to the call's: what is done once for all modes (packing and sorting the coordinates, about
    a third of this build) has its share in each.  The part outside them is one sum over the values."""
    rng = np.random.default_rng(3)
    dims, nnz = (300, 300, 30_000), 1_500_000
    inds = [np.minimum(d * rng.random(nnz) ** 2, d - 1).astype(np.uint32) for d in dims]
    vals = rng.uniform(-1, 1, nnz).astype(np.float32)
    share = 0.0
    for _ in range(5):
        begin = time.perf_counter()
        h = B.build_format(dims, inds, vals)
        call = time.perf_counter() - begin
        share = max(share, sum(B.get_stats(h, m)["build_seconds"] for m in range(3)) / call)
        assert share <= 1.0
        B.free(h)
    assert share >= 0.9


_PEAK = """
import numpy as np
from paper_1904_03329_amd import binding as B
def kib(field):
    with open("/proc/self/status") as f:
        return [int(l.split()[1]) for l in f if l.startswith(field)][0]
rng, dims, nnz = np.random.default_rng(2), {dims}, {nnz}
inds = [rng.integers(0, d, size=nnz, dtype=np.uint32) for d in dims]
vals = rng.random(nnz, dtype=np.float32)
B.free(B.build_format(dims, [i[:100] for i in inds], vals[:100]))
before = kib("VmRSS:")
h = B.build_format(dims, inds, vals)
print((kib("VmHWM:") - before) * 1024 / nnz, B.device_bytes(h) / nnz)
"""


@pytest.mark.parametrize("dims", [(300, 300, 30_000), (30_000, 300, 300), (300, 30_000, 300)])
def test_peak_memory_of_a_build(dims):
    """Beside the format itself the build holds one sorted pair of key and value (12 bytes a nonzero) in its last fill;
    the pairs other modes were sorted in are gone.  20 bytes a nonzero leave room for tables and what the allocator keeps;
    the two pairs more that a builder without releases holds are 24."""
    out = subprocess.run([sys.executable, "-c", _PEAK.format(dims=dims, nnz=9_000_000)], capture_output=True, text=True,
                         check=True, cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    peak, formats = map(float, out.stdout.split()[-2:])
    print(f"{dims}: peak {peak:.1f}, format {formats:.1f} bytes a nonzero")
    assert peak <= formats + 20
