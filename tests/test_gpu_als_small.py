"""The mode update's R x R algebra and tile kernels at their edges: rank-deficient products of Gram matrices (the eigenvalue
form) and matrices that end inside a tile or inside one row of 32 floats, against the numpy fp64 oracle."""
import numpy as np
import pytest

from oracle import cpd_als

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lazy", [False, True])
@pytest.mark.parametrize("rank", [8, 16, 32, 64, 128])
def test_rank_deficient_update(rank, lazy):
    """Two identical components: V has two equal rows, so the update takes the pseudo-inverse."""
    import torch
    from paper_1904_03329_amd import CpdAls, HbcsfTensor

    rng = np.random.default_rng(rank)
    dims = (300, 301, 157)
    flat = rng.choice(int(np.prod(dims)), size=30000, replace=False)
    inds = [(flat // (dims[1] * dims[2])).astype(np.uint32), (flat // dims[2] % dims[1]).astype(np.uint32),
            (flat % dims[2]).astype(np.uint32)]
    vals = rng.uniform(0.1, 1.0, size=flat.size).astype(np.float32)
    facs = [rng.uniform(-1, 1, size=(d, rank)).astype(np.float32) for d in dims]
    for f in facs:
        f[:, 1] = f[:, 0]
    t = HbcsfTensor(dims, inds, vals).to_device()
    als = CpdAls(t, rank)
    dfacs = [torch.from_numpy(f.copy()).cuda() for f in facs]
    print("als deficient", rank, lazy, flush=True)
    fit = als.iteration(dfacs, lazy=lazy)
    als.normalise(dfacs)
    want, lam = cpd_als.als_iteration(dims, inds, vals, facs)
    # the two components stay equal up to rounding, so what the later updates invert has one singular value at rounding
    # level: the model is compared, not the factors
    got = [f.cpu().numpy() for f in dfacs]
    model = cpd_als.model_values(inds, got, als.lam.cpu().numpy())
    ref = cpd_als.model_values(inds, want, lam)
    assert np.max(np.abs(model - ref)) <= 2e-3 * np.max(np.abs(ref))
    assert abs(fit - cpd_als.fit(dims, inds, vals, want, lam)) <= 1e-3
    als.close()
    t.close()


def _nearly_equal_columns(rank, eps):
    """A third of a rank-4 tensor's entries, and starting factors whose first two columns differ by eps."""
    rng = np.random.default_rng(rank)
    dims = (16, 12, 6007)
    flat = rng.choice(int(np.prod(dims)), size=380_000, replace=False)
    inds = [x.astype(np.uint32) for x in np.unravel_index(flat, dims)]
    vals = cpd_als.model_values(inds, [rng.uniform(0, 1, size=(d, 4)) for d in dims], np.ones(4)).astype(np.float32)
    facs = [rng.uniform(0, 1, size=(d, rank)).astype(np.float32) for d in dims]
    for f in facs:
        f[:, 1] = f[:, 0] + eps * rng.uniform(-1, 1, f.shape[0]).astype(np.float32)
    return dims, inds, vals, facs


@pytest.mark.parametrize("eps", [1.0, 1e-3])
@pytest.mark.parametrize("rank", [8, 16, 32, 64, 128])
def test_fit_of_a_put_off_update_is_that_of_the_factors_written(rank, eps):
    """||model||^2 is the sum of V's entries times those of the last factor's Gram matrix.  Its entries are fp32 sums of 128
    rows at most (each added with one rounding of up to 2^-24, as a random walk sqrt(128) / 3 of them): 2^-22 of the
    terms' magnitudes bounds the error, and the residual's with it.  An inner product taken from the same sum, as if the
    factor solved the normal equations exactly, is off by several times that."""
    import torch
    from paper_1904_03329_amd import CpdAls, HbcsfTensor

    dims, inds, vals, facs = _nearly_equal_columns(rank, eps)
    t = HbcsfTensor(dims, inds, vals).to_device()
    als = CpdAls(t, rank)
    dfacs = [torch.from_numpy(f.copy()).cuda() for f in facs]
    print("als fit", rank, eps, flush=True)
    fit = als.iteration(dfacs, lazy=True)
    got = [f.cpu().numpy() for f in dfacs]   # not normalised yet: the model without weights
    want = cpd_als.fit(dims, inds, vals, got, np.ones(rank))
    terms = np.abs(np.prod([cpd_als.gram(f) for f in got], axis=0)).sum() / np.sum(vals.astype(np.float64) ** 2)
    print(f"fit {fit:.8f}, off by {fit - want:+.1e}, terms {terms:.1f}", flush=True)
    assert abs(fit - want) <= 2.0 ** -22 * (1 + terms) / (2 * (1 - want))
    als.close()
    t.close()


def _one_small_pivot(rank, ratio):
    """Factors with nearly orthogonal columns, one of them scaled so that its pivot in V is about `ratio` of the largest
    diagonal entry: V = D (I + E) D with a well conditioned I + E, so that the update is well determined all the same."""
    rng = np.random.default_rng(rank)
    dims = (333, 4 * rank + 5, 4 * rank + 9)
    flat = rng.choice(int(np.prod(dims)), size=20_000, replace=False)
    inds = [x.astype(np.uint32) for x in np.unravel_index(flat, dims)]
    vals = rng.uniform(0.1, 1.0, size=flat.size).astype(np.float32)
    facs = []
    for d in dims:
        f = rng.normal(size=(d, rank))
        f /= np.linalg.norm(f, axis=0)
        f[:, rank // 2 + 1] *= ratio ** 0.25
        facs.append(f.astype(np.float32))
    return dims, inds, vals, facs


@pytest.mark.parametrize("lazy", [False, True])
@pytest.mark.parametrize("ratio", [5e-11, 2e-10])
@pytest.mark.parametrize("rank", [8, 16, 32, 64, 128])
def test_pivots_on_both_sides_of_the_line(oracle, rank, ratio, lazy):
    """A pivot below 1e-10 of the largest diagonal entry sends the update from the sweep to the eigenvalue form.  Both give
    A = M V^-1, whose entries are sums of n rows' terms and R products in fp32: gamma (|M| |P|) bounds their error, with |M|
    the MTTKRP of the absolute values and gamma = 2^-24 times the operations in one entry's chain."""
    import torch
    from paper_1904_03329_amd import CpdAls, HbcsfTensor

    dims, inds, vals, facs = _one_small_pivot(rank, ratio)
    v = cpd_als.gram(facs[1]) * cpd_als.gram(facs[2])
    pivots = np.diag(np.linalg.cholesky(v)) ** 2
    assert (pivots.min() < 1e-10 * v.max()) == (ratio < 1e-10)
    p = np.linalg.inv(v)
    want = oracle.mttkrp(dims, inds, vals, facs, 0) @ p
    most = np.abs(oracle.mttkrp(dims, inds, np.abs(vals), [np.abs(f) for f in facs], 0)) @ np.abs(p)
    bound = 2.0 ** -24 * (np.bincount(inds[0]).max() + rank + 8) * most
    norm = np.linalg.norm(want, axis=0)
    t = HbcsfTensor(dims, inds, vals).to_device()
    als = CpdAls(t, rank)
    dfacs = [torch.from_numpy(f.copy()).cuda() for f in facs]
    print("als pivot", rank, ratio, lazy, flush=True)
    als.iteration(dfacs, lazy=lazy)
    assert ratio > 1e-10 or als.phase_ms()[2] > 0   # the eigenvalue form was taken, also after a sweep beside the MTTKRP
    got = dfacs[0].cpu().numpy().astype(np.float64)
    got /= np.linalg.norm(got, axis=0)
    want /= norm
    bound = bound / norm + np.abs(want) * (np.linalg.norm(bound, axis=0) / norm)
    print(f"largest error / bound {np.max(np.abs(got - want) / bound):.3f}", flush=True)
    assert np.all(np.abs(got - want) <= bound)
    als.close()
    t.close()


def _one_infinite_value(rank):
    rng = np.random.default_rng(rank)
    dims = (100, 61, 37)
    flat = rng.choice(int(np.prod(dims)), size=2000, replace=False)
    inds = [x.astype(np.uint32) for x in np.unravel_index(flat, dims)]
    vals = rng.uniform(0.1, 1.0, size=flat.size).astype(np.float32)
    vals[np.flatnonzero(inds[0] == 41)[0]] = np.inf
    return dims, inds, vals, [rng.uniform(-1, 1, size=(d, rank)).astype(np.float32) for d in dims]


@pytest.mark.parametrize("lazy", [False, True])
@pytest.mark.parametrize("rank", [8, 16, 32, 64, 128])
def test_pseudo_inverse_of_a_matrix_that_is_not_finite(rank, lazy):
    """An infinite value makes one row of the first factor infinite or NaN, hence its Gram matrix and the V of both later
    updates: no row of theirs can come out finite."""
    import torch
    from paper_1904_03329_amd import CpdAls, HbcsfTensor

    dims, inds, vals, facs = _one_infinite_value(rank)
    t = HbcsfTensor(dims, inds, vals).to_device()
    als = CpdAls(t, rank)
    dfacs = [torch.from_numpy(f.copy()).cuda() for f in facs]
    print("als not finite", rank, lazy, flush=True)
    als.iteration(dfacs, lazy=lazy)
    for m in (1, 2):
        assert bool((~torch.isfinite(dfacs[m])).any(dim=1).all()), f"factor {m}"
    als.close()
    t.close()


@pytest.mark.parametrize("rank", [8, 16, 64, 128])
@pytest.mark.parametrize("rows", [1, 3, 33, 129, 4099])
def test_gram_of_ragged_matrices(rank, rows):
    import torch
    from paper_1904_03329_amd import binding as B

    a = np.random.default_rng(rows).uniform(-1, 1, size=(rows, rank)).astype(np.float32)
    # the matrix ends where its allocation does not: what follows must not be taken in
    buf = torch.full((rows * rank + 64,), 1e30, device="cuda")
    buf[:rows * rank] = torch.from_numpy(a.reshape(-1)).cuda()
    ws = torch.empty(B.gram_workspace_bytes(rank), dtype=torch.uint8, device="cuda")
    s = torch.full((rank, rank), float("nan"), dtype=torch.float64, device="cuda")
    B.gram(buf.data_ptr(), rows, rank, ws.data_ptr(), ws.numel(), s.data_ptr(), torch.cuda.current_stream().cuda_stream)
    want = cpd_als.gram(a)
    assert np.max(np.abs(s.cpu().numpy() - want)) <= 1e-5 * np.max(np.abs(want))
