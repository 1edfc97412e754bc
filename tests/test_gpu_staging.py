"""GPU parity where a unit's staging has edges: streams that end inside a 16-byte load, inside a part or one nonzero beyond a
unit, fiber segments that fill or straddle a lane's four, and more slices than one load brings."""
import numpy as np
import pytest

import gpu_util as GU

pytestmark = pytest.mark.gpu


def _tensor(dims, nnz, fiber, seed):
    """nnz nonzeros with distinct coordinates, `fiber` consecutive leaves under each fiber (the last one cut)."""
    rng = np.random.default_rng(seed)
    fibers = -(-nnz // fiber)
    cells = rng.choice(int(np.prod(dims[:-1])), size=fibers, replace=False)
    upper = np.stack(np.unravel_index(cells, dims[:-1])).repeat(fiber, axis=1)[:, :nnz]
    leaf = (rng.integers(0, dims[-1], fibers).repeat(fiber)[:nnz] + np.tile(np.arange(fiber), fibers)[:nnz]) % dims[-1]
    inds = [np.ascontiguousarray(x, dtype=np.uint32) for x in (*upper, leaf)]
    return inds, rng.uniform(-1, 1, nnz).astype(np.float32)


@pytest.mark.parametrize("rank, dtype", [(8, np.float32), (32, np.float32), (128, np.float32), (32, np.float64)])
@pytest.mark.parametrize("dims", [(13, 90, 70), (11, 20, 9, 70), (7, 8, 5, 6, 70)])
@pytest.mark.parametrize("nnz, fiber", [(1, 1), (63, 1), (257, 1), (515, 3), (1021, 5), (255, 64), (1029, 64)])
def test_ends_of_the_stream(oracle, rank, dtype, dims, nnz, fiber):
    inds, vals = _tensor(dims, nnz, fiber, seed=nnz + fiber)
    rng = np.random.default_rng(7)
    facs = [rng.uniform(0, 1, (d, rank)).astype(dtype) for d in dims]
    ref, tol = (oracle.mttkrp_f64, GU.REL_TOL_F64) if dtype == np.float64 else (oracle.mttkrp, GU.REL_TOL)
    for opts in (dict(), dict(group_mask=4), dict(fiber_threshold=8)):
        outs, _ = GU.gpu_mttkrp_all_modes(dims, inds, vals, facs, **opts)
        for mode, out in enumerate(outs):
            GU.assert_close(out, ref(dims, inds, vals, facs, mode), f"{opts} mode {mode}", tol)


@pytest.mark.parametrize("dims", [(4000, 3, 50), (2000, 3, 2, 50)])
def test_many_slices_in_a_unit(oracle, dims):
    """Slices of two nonzeros: 256 of them in a unit of 512, more than the two loads of 64 that are issued together."""
    inds, vals = _tensor(dims, 2 * (dims[0] // 2), 2, seed=3)
    inds[0] = np.arange(len(vals), dtype=np.uint32) // 2   # two nonzeros a slice, one fiber each
    for m in range(1, len(dims) - 1):
        inds[m][:] = inds[m][::2].repeat(2)
    rng = np.random.default_rng(1)
    facs = [rng.uniform(0, 1, (d, 32)).astype(np.float32) for d in dims]
    for steps in (0, 8):
        outs, _ = GU.gpu_mttkrp_all_modes(dims, inds, vals, facs, tune_steps=steps, group_mask=4)
        for mode, out in enumerate(outs):
            GU.assert_close(out, oracle.mttkrp(dims, inds, vals, facs, mode), f"steps {steps} mode {mode}")
