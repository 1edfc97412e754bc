"""GPU parity of the B-CSF kernels' fiber-row loads: how many fibers end within four steps of a lane group (none, one, all
four), at orders 3 (deepest level) and 4 (the level above it), with 4 and, at rows of 128 bytes, 8 gathers in flight."""
import numpy as np
import pytest

import gpu_util as GU

pytestmark = pytest.mark.gpu


def _tensor(order, lengths, nnz, seed):
    """Fibers of the given lengths one after the other: at order 3 deepest-level ones, at order 4 level-1 ones with
    deepest-level fibers of two nonzeros inside."""
    rng = np.random.default_rng(seed)
    n = np.resize(np.asarray(lengths), nnz)
    fiber = np.repeat(np.arange(n.size), n)[:nnz]
    place = np.arange(nnz) - np.searchsorted(fiber, fiber)
    per = rng.integers(1, 30)  # fibers per slice
    cols = [fiber // per, fiber % per] + ([place // 2, place % 2] if order == 4 else [place])
    dims = [int(c.max()) + 1 + 3 * (i == 0) for i, c in enumerate(cols)]
    vals = rng.uniform(-1, 1, nnz).astype(np.float32)
    return tuple(dims), [c.astype(np.uint32) for c in cols], vals


@pytest.mark.parametrize("rank, dtype", [(8, np.float32), (16, np.float32), (32, np.float32), (64, np.float32),
                                         (128, np.float32), (16, np.float64), (32, np.float64)])
@pytest.mark.parametrize("order", [3, 4])
@pytest.mark.parametrize("lengths", [(1,), (1, 2, 1, 5, 3, 1, 1, 9), (3,), (70,)])
def test_fiber_ends_per_block(oracle, rank, dtype, order, lengths):
    dims, inds, vals = _tensor(order, lengths, 6_007, seed=rank + order)
    rng = np.random.default_rng(3)
    facs = [rng.uniform(0, 1, size=(d, rank)).astype(dtype) for d in dims]
    ref = oracle.mttkrp_f64 if dtype == np.float64 else oracle.mttkrp
    want = [ref(dims, inds, vals, facs, mode) for mode in range(order)]
    for steps in (None, 8) if rank * np.dtype(dtype).itemsize == 128 else (None,):
        # plain B-CSF (single nonzeros too are slices and fibers of the one group), levels in their natural order
        outs, _ = GU.gpu_mttkrp_all_modes(dims, inds, vals, facs, tune_steps=steps, group_mask=4, mode_order_policy=2)
        for mode in range(order):
            GU.assert_close(outs[mode], want[mode], f"order {order} rank {rank} lengths {lengths} mode {mode} steps {steps}",
                            GU.REL_TOL_F64 if dtype == np.float64 else GU.REL_TOL)
