"""The host builder's count of distinct rows each group gathers, per tree level: lengths around the 64 indices that are looked
at together, one nonzero, rows that nearly all nonzeros share, and the sorted form for long modes."""
import numpy as np
import pytest

from paper_1904_03329_amd import binding as B


@pytest.mark.parametrize("nnz", [1, 63, 64, 65, 129, 20_000])
@pytest.mark.parametrize("dims", [(9, 300, 50), (2000, 7, 30, 11), (500, 1 << 20, 40)])
@pytest.mark.parametrize("opts", [dict(), dict(group_mask=4), dict(mode_order_policy=1)])
def test_distinct_rows(dims, nnz, opts):
    rng = np.random.default_rng(nnz)
    flat = rng.choice(int(np.prod(dims)), size=min(nnz, int(np.prod(dims)) // 2), replace=False)
    if nnz > 1000:
        flat = np.unique(flat // 3)   # runs of neighbours: fibers and slices of many nonzeros
    inds = [x.astype(np.uint32) for x in np.unravel_index(flat, dims)]
    h = B.build_format(dims, inds, np.ones(len(flat), dtype=np.float32), **opts)
    try:
        for mode in range(len(dims)):
            st = B.get_stats(h, mode)
            for g in range(3):
                for level in range(1, len(dims)):
                    ind = B.host_array(h, mode, g, level, B.ARR_IND)
                    if g == B.GROUP_CSF and level < len(dims) - 1:
                        ind = ind[:-1]   # closed by one entry more
                    assert st["distinct_rows"][g][level] == len(np.unique(ind)), (mode, g, level)
    finally:
        B.free(h)
