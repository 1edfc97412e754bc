"""What the host builder refuses, what it reports and what it holds (no GPU)."""
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
