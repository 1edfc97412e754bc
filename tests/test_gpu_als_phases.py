"""The phase times of a CPD-ALS iteration where the pseudo-inverse runs in the MTTKRP's launch: every kernel counts to the
phase it belongs to, as it does where the launches are separate."""
import numpy as np
import pytest

from oracle import cpd_als

pytestmark = pytest.mark.gpu


def _phases(dims, inds, vals, facs, profiled, iterations=4):
    """The smallest of a few iterations' phase times, the last ones' fit; profiled launches are taken one by one."""
    import torch
    from paper_1904_03329_amd import CpdAls, HbcsfTensor, binding as B

    t = HbcsfTensor(dims, inds, vals).to_device()
    if profiled:
        B.tune(t.handle, B.TUNE_PROFILE, 4)
    als = CpdAls(t, facs[0].shape[1])
    ms = []
    for _ in range(iterations):
        work = [torch.from_numpy(f).cuda() for f in facs]
        als.iteration(work, lazy=True)
        ms.append(als.phase_ms())
    als.close()
    t.close()
    best = [min(m[k] for m in ms) for k in range(4)]
    print(dims, facs[0].shape[1], "profiled" if profiled else "in one launch", best, flush=True)
    return best


def _tensor(dims, nnz, seed):
    rng = np.random.default_rng(seed)
    flat = rng.choice(int(np.prod(dims)), size=nnz, replace=False)
    inds = [x.astype(np.uint32) for x in np.unravel_index(flat, dims)]
    return rng, inds, rng.uniform(-1, 1, nnz).astype(np.float32)


@pytest.mark.parametrize("long_mode", [0, 1])
def test_output_definition_is_mttkrp_time(long_mode):
    """Three million output rows of 128 bytes and few nonzeros: writing the rows is nearly all of the MTTKRP (384 MB, 50 us at
    8 TB/s, where the rest takes 10 to 20 us), so without it less than half of its time would be left."""
    dims = [41, 23, 29]
    dims[long_mode] = 3_000_000
    rng, inds, vals = _tensor(tuple(dims), 60_000, 2)
    facs = [rng.uniform(-1, 1, (d, 32)).astype(np.float32) for d in dims]
    beside, alone = (_phases(dims, inds, vals, facs, p) for p in (False, True))
    assert beside[0] > 0.5 * alone[0]
    assert beside[2] == 0 and alone[2] > 0


def test_eigenvalue_form_is_inverse_time():
    """Two equal columns: every update takes the eigenvalue form, several hundred microseconds at rank 64 beside an MTTKRP of
    some ten."""
    dims, rank = (300, 301, 157), 64
    rng, inds, vals = _tensor(dims, 30_000, 3)
    facs = [rng.uniform(-1, 1, (d, rank)).astype(np.float32) for d in dims]
    for f in facs:
        f[:, 1] = f[:, 0]
    v = np.prod([cpd_als.gram(f) for f in facs[1:]], axis=0)
    assert np.linalg.matrix_rank(v) < rank
    beside, alone = (_phases(dims, inds, vals, facs, p) for p in (False, True))
    assert beside[2] > 0.5 * alone[2] and beside[2] > beside[0]


@pytest.mark.parametrize("rank", [8, 16, 32])
def test_mttkrp_keeps_its_time_beside_the_eigenvalue_form(rank):
    """Two equal columns and four million nonzeros: up to rank 32 the eigenvalue form runs in the launch of an MTTKRP that takes
    tens of microseconds.  That launch's time up to its last blocks is MTTKRP time, the same as without equal columns (the form
    begins some microseconds into it: counted from there, most of the MTTKRP would be missing)."""
    dims = (400, 300, 250)
    rng, inds, vals = _tensor(dims, 4_000_000, 4)
    facs = [rng.uniform(-1, 1, (d, rank)).astype(np.float32) for d in dims]
    regular = _phases(dims, inds, vals, facs, False)
    for f in facs:
        f[:, 1] = f[:, 0]
    equal = _phases(dims, inds, vals, facs, False)
    assert regular[2] == 0 and equal[2] > 0
    assert 0.7 * regular[0] < equal[0] < 1.5 * regular[0]
