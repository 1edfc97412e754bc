"""The pseudo-inverse of a put-off ALS update runs in a block of the MTTKRP launch where that takes one (rank <= 64), and in
a launch before it elsewhere; a profiled tensor's launches are taken one by one, so it goes the other way."""
import numpy as np
import pytest

from oracle import cpd_als

pytestmark = pytest.mark.gpu


def _problem(dims, nnz, rank):
    rng = np.random.default_rng(rank + len(dims))
    nnz = min(nnz, int(np.prod(dims)) // 2)
    flat = rng.choice(int(np.prod(dims)), size=nnz, replace=False)
    inds = [x.astype(np.uint32) for x in np.unravel_index(flat, dims)]
    vals = rng.uniform(-1, 1, nnz).astype(np.float32)
    return inds, vals, [rng.uniform(-1, 1, (d, rank)).astype(np.float32) for d in dims]


def _v(facs, n):
    return np.prod([cpd_als.gram(f) for m, f in enumerate(facs) if m != n], axis=0)


def _iterate(dims, inds, vals, facs, opts, profiled):
    """One iteration: the factors as they are written, then normalised with lambda and the fit, the phase times, the groups
    that some mode has."""
    import torch
    from paper_1904_03329_amd import CpdAls, HbcsfTensor, binding as B

    t = HbcsfTensor(dims, inds, vals, **opts).to_device()
    if profiled:
        B.tune(t.handle, B.TUNE_PROFILE, 4)
    als = CpdAls(t, facs[0].shape[1])
    work = [torch.from_numpy(f).cuda() for f in facs]
    print("als beside", dims, facs[0].shape[1], "profiled" if profiled else "in one launch", flush=True)
    fit = als.iteration(work, lazy=True)
    ms = als.phase_ms()
    written = [w.cpu().numpy() for w in work]
    als.normalise(work)
    done = [w.cpu().numpy() for w in work] + [als.lam.cpu().numpy(), np.array([fit, 1.0])]   # the fit's scale is 1
    groups = [set(g for g in range(3) if t.stats(m)["group_nnz"][g]) for m in range(len(dims))]
    als.close()
    t.close()
    return written, done, ms, groups


@pytest.mark.parametrize("rank", [8, 16, 32, 64, 128])
@pytest.mark.parametrize("dims, nnz, opts, groups", [
    ((300, 200, 90), 30_000, {}, {2}),
    ((4000, 40, 30), 30_000, {}, {0, 1, 2}),             # CSL and B-CSF in one launch
    ((5000, 4000, 3000), 6000, {}, {0, 1}),
    ((90, 60, 40, 20), 300_000, {}, {2}),                # order 4, units of 256 nonzeros
    ((60, 50, 20, 13, 11), 40_000, {}, {2}),             # order 5
])
def test_same_result_beside_and_before(rank, dims, nnz, opts, groups):
    inds, vals, facs = _problem(dims, nnz, rank)
    # the sweep is the same code; shared rows of the MTTKRP are added in an order that changes from call to call, a few
    # fp32 roundings (2^-24 each) of a row, amplified by the condition of V in the updates so far: measured against
    # itself, not against the way
    step, conds = [f.astype(np.float64) for f in facs], []
    for n in range(len(dims)):
        v = _v(step, n)
        conds.append(np.linalg.cond(v))
        step[n] = cpd_als.mttkrp(dims, inds, vals, step, n) @ np.linalg.inv(v)
    tol = 1e-6 * max(10.0, max(conds))
    print("conditions of V", [f"{c:.1f}" for c in conds], flush=True)
    assert tol <= 1e-2
    (_, a, beside, have), (_, b, before, _) = (_iterate(dims, inds, vals, facs, opts, p) for p in (False, True))
    assert any(h >= groups for h in have)
    assert (beside[2] == 0) == (rank <= 64) and before[2] > 0
    for x, y in zip(a, b):
        assert np.all(np.isfinite(x)) and np.abs(x - y).max() <= tol * np.abs(y).max()


@pytest.mark.parametrize("rank", [8, 16, 32, 64, 128])
def test_singular_matrix_beside_and_before(rank):
    """Two equal components: the sweep fails and the eigenvalue form follows, also where the sweep ran beside the MTTKRP of CSL
    and B-CSF groups.  The factor is not determined, but the model it gives with the other factors as they were is; its
    error is that of the sums in fp32 (2^-24 a term), amplified by the condition of V on its range."""
    dims = (4000, 40, 30)
    inds, vals, facs = _problem(dims, 30_000, rank)
    for f in facs:
        f[:, 1] = f[:, 0]
    f64 = [f.astype(np.float64) for f in facs]
    rows = np.einsum("jr,kr->jkr", f64[1], f64[2]).reshape(-1, rank)
    w = np.linalg.eigvalsh(_v(facs, 0))
    assert w[0] < 1e-12 * w[-1] < 1e-3 * w[1]
    want = cpd_als.mttkrp(dims, inds, vals, f64, 0) @ np.linalg.pinv(_v(facs, 0)) @ rows.T
    tol = 1e-6 * max(10.0, w[-1] / w[1])
    for profiled in (False, True):
        written, _, ms, _ = _iterate(dims, inds, vals, facs, {}, profiled)
        error = np.abs(written[0].astype(np.float64) @ rows.T - want).max() / np.abs(want).max()
        print(f"condition on the range {w[-1] / w[1]:.1f}, largest error {error:.1e}", flush=True)
        assert ms[2] > 0 and error <= tol


@pytest.mark.parametrize("rank", [8, 16, 32, 64])
@pytest.mark.parametrize("dims, nnz", [((4000, 40, 30), 30_000), ((90, 60, 40, 20), 300_000), ((60, 50, 20, 13, 11), 40_000)])
@pytest.mark.parametrize("equal", [False, True])
def test_same_result_on_another_stream(rank, dims, nnz, equal):
    """There the output is defined in a launch of its own and the launch that carries the inverse is the form that does not ask for
    rows.  Both are held to the update of mode 0 in fp64 (as above: through the model, which two equal components leave
    determined)."""
    import torch

    inds, vals, facs = _problem(dims, nnz, rank)
    if equal:
        for f in facs:
            f[:, 1] = f[:, 0]
    f64 = [f.astype(np.float64) for f in facs]
    rows = f64[1]
    for f in f64[2:]:
        rows = (rows[:, None, :] * f[None, :, :]).reshape(-1, rank)
    v = _v(facs, 0)
    w = np.linalg.eigvalsh(v)
    tol = 1e-6 * max(10.0, w[-1] / w[1 if equal else 0])
    rows = rows[np.random.default_rng(1).choice(len(rows), 2000)] if len(rows) > 2000 else rows
    want = cpd_als.mttkrp(dims, inds, vals, f64, 0) @ np.linalg.pinv(v) @ rows.T
    for stream in (torch.cuda.current_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            written, _, ms, _ = _iterate(dims, inds, vals, facs, {}, False)
        error = np.abs(written[0].astype(np.float64) @ rows.T - want).max() / np.abs(want).max()
        print(f"stream {stream.cuda_stream}: condition {tol * 1e6:.1f}, largest error {error:.1e}", flush=True)
        assert (ms[2] > 0) == equal and error <= tol
