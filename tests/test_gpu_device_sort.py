"""The device builder's pair sort (csrc/hbcsf_sort.h) at the edges of its tiles and digits: the built arrays are the host
builder's, whose sort is stable too, so equal coordinates must keep their order."""
import numpy as np
import pytest
import torch  # noqa: F401  (its libraries have to be there before the package's)

from paper_1904_03329_amd import binding as B
from test_gpu_device_build import _device_tensor, _random, _skewed, assert_same_format

pytestmark = pytest.mark.gpu

SHORT, LONG, LONG_FROM = 2048, 8192, 1 << 20   # nonzeros of a tile, and from how many on the long one is taken


@pytest.mark.parametrize("nnz", [1, 2, 63, 64, 65, 511, 513, SHORT - 1, SHORT, SHORT + 1, 5 * SHORT + 77, 40 * SHORT])
def test_short_tiles(nnz):
    dims = (300, 41, 129)
    inds, vals = _random(np.random.default_rng(nnz), dims, nnz, distinct=False)
    assert_same_format(dims, inds, vals).close()


@pytest.mark.parametrize("nnz", [LONG_FROM - 1, LONG_FROM, LONG_FROM + 1, LONG_FROM + LONG - 1, LONG_FROM + LONG + 300])
def test_where_the_tiles_change(nnz):
    dims = (700, 1025, 90)
    inds, vals = _random(np.random.default_rng(nnz), dims, nnz, distinct=False)
    assert_same_format(dims, inds, vals).close()


@pytest.mark.parametrize("dims, opts", [
    ((2, 3, 5), {}),                                             # digits of one to three bits
    ((1 << 21, 1 << 22, 1 << 21), {}),                           # all 64 bits
    ((1, 1, 1), {}), ((1, 70_000, 2), {}),
    ((3000, 2900, 2800, 2700, 2600), {}),                        # 16 passes
    ((3000, 2900, 2800, 2700, 2600), {"mid_blocking": 9}),       # 26
    ((257, 4000, 65_537, 300), {"mid_blocking": 5}),
])
@pytest.mark.parametrize("nnz", [3 * SHORT + 5, LONG_FROM + 3 * LONG + 5])
def test_widths(dims, opts, nnz):
    inds, vals = _random(np.random.default_rng(3), dims, nnz, distinct=False)
    assert_same_format(dims, inds, vals, **opts).close()


@pytest.mark.parametrize("nnz", [30_000, LONG_FROM + 12_345])
def test_one_digit_holds_nearly_all(nnz):
    """Every digit of a mode the same but for a few nonzeros, sorted and reversed input."""
    dims = (70_000, 300, 400)
    rng = np.random.default_rng(nnz)
    inds, vals = _random(rng, dims, nnz, distinct=False)
    inds[0][rng.random(len(vals)) < 0.999] = 65_535
    inds[1][:] = 255
    assert_same_format(dims, inds, vals).close()
    up = np.lexsort((inds[2], inds[1], inds[0]))
    for order in (up, up[::-1]):
        assert_same_format(dims, [x[order] for x in inds], vals[order]).close()


def test_skewed():
    dims = (5000, 900, 130, 70)
    inds, vals = _skewed(np.random.default_rng(5), dims, 1_500_000)
    assert_same_format(dims, inds, vals).close()


@pytest.mark.parametrize("nnz", [SHORT + 1, LONG_FROM + 1])
def test_bad_index_in_the_last_tile(nnz):
    dims = (300, 41, 129)
    inds, vals = _random(np.random.default_rng(1), dims, nnz, distinct=False)
    inds[2][-1] = 2 ** 32 - 1
    with pytest.raises(B.HbcsfError, match="below its dimension"):
        _device_tensor(dims, inds, vals)
