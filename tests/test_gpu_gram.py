"""GPU parity of hbcsf_gram (the Gram matrices A^T A of Eq. 3) against the fp64 oracle.

Bar: the device multiplies in fp32 and keeps fp32 partial sums for at most 128 rows (rank 32; 32 at the other ranks)
before they go to fp64, so an entry's error is bounded by 128 * 2^-24 * sum_i |A[i][r] A[i][s]| <= 7.7e-6 * max(diag S)
(Cauchy-Schwarz); the test asks for max |S_gpu - S_oracle| <= 1e-5 * max |S_oracle|.
"""
import numpy as np
import pytest

from oracle import cpd_als
from paper_1904_03329_amd import binding as B

pytestmark = pytest.mark.gpu

TOL = 1e-5


def _gram(a, workspace_bytes=None, prefill=None):
    import torch

    rows, rank = a.shape
    da = torch.from_numpy(a).cuda()
    n = B.gram_workspace_bytes(rank) if workspace_bytes is None else workspace_bytes
    ws = torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")
    if prefill is not None:
        ws.view(torch.float64).fill_(prefill)
    s = torch.full((rank, rank), float("nan"), dtype=torch.float64, device="cuda")
    B.gram(da.data_ptr() if rows else ws.data_ptr(), rows, rank, ws.data_ptr(), n, s.data_ptr(),
           torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return s.cpu().numpy()


@pytest.mark.parametrize("rank", [32, 8, 16, 64, 128])
@pytest.mark.parametrize("rows", [1, 31, 1000, 100_003])
def test_gram_matches_the_oracle(rank, rows):
    rng = np.random.default_rng(rank * 1000 + rows % 997)
    a = rng.uniform(-1, 1, size=(rows, rank)).astype(np.float32)
    print("gram", rows, rank, flush=True)
    want = cpd_als.gram(a)
    got = _gram(a, prefill=float("nan"))          # stale scratch contents must not matter
    assert np.all(np.isfinite(got))
    assert np.max(np.abs(got - want)) <= TOL * np.max(np.abs(want))
    assert np.array_equal(got, _gram(a, prefill=3.0)), "equal inputs must give equal bits"


def test_gram_large_positive_matrix_and_small_workspace():
    """A 3 M-row matrix of positive entries (every wavefront chunk is many flush periods long), with the full
    workspace and with one that holds a single slot (one workgroup does all rows)."""
    rng = np.random.default_rng(5)
    a = rng.uniform(0, 1, size=(3_000_000, 32)).astype(np.float32)
    want = cpd_als.gram(a)
    print("gram large", flush=True)
    for nbytes in (None, 32 * 32 * 8, 5 * 32 * 32 * 8 + 100):
        got = _gram(a, workspace_bytes=nbytes)
        assert np.max(np.abs(got - want)) <= TOL * np.max(np.abs(want)), nbytes


@pytest.mark.parametrize("rank", [8, 16, 64, 128])
def test_fp32_sums_end_after_32_rows(rank):
    """At these ranks no fp32 sum goes over more than 32 rows (of a residue class modulo 32 / rank below rank 32).  The
    first such stretch sums to 2^26, the next three to 32 each: in fp32 2^26 + 2 is 2^26 again, so a sum over two of the
    stretches would lose every one of the small products; taken apart all sums are exact."""
    rows = 32 * max(1, 32 // rank)
    a = np.ones((4 * rows, rank), np.float32)
    a[:rows] = 0
    a[:max(1, 32 // rank)] = 8192
    assert np.array_equal(_gram(a), cpd_als.gram(a))


def test_gram_of_no_rows_is_zero_and_errors():
    import torch

    assert np.array_equal(_gram(np.zeros((0, 16), np.float32), prefill=float("nan")), np.zeros((16, 16)))
    a = torch.zeros((64, 32), device="cuda")
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    s = torch.zeros((32, 32), dtype=torch.float64, device="cuda")
    for args, code in (((a.data_ptr(), 64, 24, ws.data_ptr(), ws.numel(), s.data_ptr()), -1),     # rank
                       ((0, 64, 32, ws.data_ptr(), ws.numel(), s.data_ptr()), -1),                # null matrix
                       ((a.data_ptr(), 64, 32, 0, ws.numel(), s.data_ptr()), -1),                 # null workspace
                       ((a.data_ptr(), 64, 32, ws.data_ptr() + 8, ws.numel() - 8, s.data_ptr()), -1),  # alignment
                       ((a.data_ptr(), 64, 32, ws.data_ptr(), 100, s.data_ptr()), -3)):           # below one slot
        with pytest.raises(B.HbcsfError) as e:
            B.gram(*args)
        assert e.value.code == code
