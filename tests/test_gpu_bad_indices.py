"""Indices that are not below their dimension are refused by the device-side builder, also where the distinct values would
number more slices than the mode has rows (the builder's tables have room for those only)."""
import numpy as np
import pytest

from paper_1904_03329_amd import HbcsfTensor
from paper_1904_03329_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("top", [1024, 2 ** 32])
def test_more_index_values_than_rows(mode, top):
    import torch

    dims, nnz = (513, 600, 530), 20_000
    rng = np.random.default_rng(7)
    inds = [rng.integers(0, d, nnz, dtype=np.uint32) for d in dims]
    good = [x.copy() for x in inds]
    inds[mode] = rng.integers(0, top, nnz, dtype=np.uint64).astype(np.uint32)
    vals = torch.ones(nnz, device="cuda")
    dev = lambda a: [torch.from_numpy(x.view(np.int32)).cuda() for x in a]
    with pytest.raises(B.HbcsfError, match="below its dimension"):
        HbcsfTensor.from_device_coo(dims, dev(inds), vals)
    t = HbcsfTensor.from_device_coo(dims, dev(good), vals)
    out = t.mttkrp(mode, [torch.ones((d, 32), device="cuda") for d in dims])
    # ones everywhere: a row counts its nonzeros, exactly
    want = np.bincount(good[mode], minlength=dims[mode]).astype(np.float32)
    assert (out.cpu().numpy() == want[:, None]).all()
