"""The pseudo-inverse of a put-off ALS update runs in a block of the MTTKRP launch where that takes one (rank <= 64), and in
a launch before it elsewhere; a profiled tensor's launches are taken one by one, so it goes the other way."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank", [8, 16, 32, 64, 128])
@pytest.mark.parametrize("dims, nnz, opts", [
    ((300, 200, 90), 30_000, {}),                        # B-CSF group
    ((300, 4, 3), 1200, dict(mode_order_policy=1)),      # CSL and B-CSF groups
    ((5000, 4000, 3000), 6000, {}),                      # COO and CSL groups only
    ((90, 60, 40, 20), 300_000, {}),                     # order 4, units of 256 nonzeros
])
def test_same_result_beside_and_before(rank, dims, nnz, opts):
    import torch

    from paper_1904_03329_amd import CpdAls, HbcsfTensor, binding as B

    rng = np.random.default_rng(rank + len(dims))
    nnz = min(nnz, int(np.prod(dims)) // 2)
    flat = rng.choice(int(np.prod(dims)), size=nnz, replace=False)
    inds = [x.astype(np.uint32) for x in np.unravel_index(flat, dims)]
    vals = rng.uniform(-1, 1, nnz).astype(np.float32)
    facs = [rng.uniform(0, 1, (d, rank)).astype(np.float32) for d in dims]
    results = []
    for profiled in (False, True):
        t = HbcsfTensor(dims, inds, vals, **opts).to_device()
        if profiled:
            B.tune(t.handle, B.TUNE_PROFILE, 4)
        als = CpdAls(t, rank)
        work = [torch.from_numpy(f).cuda() for f in facs]
        fit = als.iteration(work, lazy=True)
        als.normalise(work)
        results.append([w.cpu().numpy() for w in work] + [als.lam.cpu().numpy(), np.array([fit])])
        als.close()
        t.close()
    # the sweep is the same code; shared rows of the MTTKRP are added in an order that changes from call to call, a few
    # fp32 roundings (2^-24 each) of a row, amplified by the condition of V: measured against itself, not against the way
    conds = [np.linalg.cond(np.prod([f.T.astype(np.float64) @ f for m, f in enumerate(facs) if m != n], axis=0))
             for n in range(len(dims))]
    tol = 1e-6 * max(10.0, max(conds))
    for a, b in zip(*results):
        assert np.all(np.isfinite(a)) and np.abs(a - b).max() <= tol * np.abs(b).max()
