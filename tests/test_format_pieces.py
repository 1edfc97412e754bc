"""The host builder cuts long slices into pieces for its threads and sorts once for all modes: slices longer than a
piece (4096 nonzeros), piece ends on and off the run grid, keys above 64 bits."""
import numpy as np
import pytest

import format_walk as FW
from paper_1904_03329_amd import binding as B


@pytest.mark.parametrize("dims, opts", [
    ((5, 300, 700), dict()),
    ((5, 300, 700), dict(hybrid_granularity=1, fiber_threshold=8)),
    ((4, 5, 90, 60), dict(mode_order_policy=1)),
    ((4, 5, 90, 60), dict(mid_blocking=2, mode_order_policy=2)),
    ((3, 1 << 22, 1 << 22, 1 << 22), dict()),
    ((3, 4, 5, 40, 50), dict(fiber_threshold=16)),
])
def test_long_slices(oracle, dims, opts):
    rng = np.random.default_rng(11)
    nnz, order = 26_001, len(dims)
    inds = [np.minimum((d * rng.random(nnz) ** 3).astype(np.uint32), d - 1).astype(np.uint32) for d in dims]
    for m in range(order):
        if dims[m] > 10_000:
            inds[m] = (inds[m] % 97) * np.uint32(dims[m] // 97)
    vals = rng.uniform(-1, 1, nnz).astype(np.float32)
    h = B.build_format(dims, inds, vals, **opts)
    try:
        for mode in range(order):
            fmt = FW.read_mode(h, mode, order)
            lm = fmt["level_mode"]
            assert sum(fmt["stats"]["group_nnz"]) == nnz
            cols, v = FW.expand_to_coo(fmt)
            got = np.stack([cols[lm.index(m)].astype(np.int64) for m in range(order)] + [v.view(np.uint32).astype(np.int64)])
            want = np.stack([x.astype(np.int64) for x in inds] + [vals.view(np.uint32).astype(np.int64)])
            assert np.array_equal(got[:, np.lexsort(got[::-1])], want[:, np.lexsort(want[::-1])])
            if max(dims) < 10_000:
                facs = [rng.uniform(0, 1, size=(d, 8)).astype(np.float32) for d in dims]
                out = FW.emulate_kernels(fmt, facs, dims[mode], 8)
                np.testing.assert_allclose(out, oracle.mttkrp(dims, inds, vals, facs, mode), rtol=1e-9, atol=1e-11)
    finally:
        B.free(h)
