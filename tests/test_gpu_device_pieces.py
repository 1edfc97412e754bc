"""Device builds into memory that is asked for piece by piece, into one arena and moved into another: the same arrays and results.
Statistics of groups that hold every nonzero, whose distinct rows are counted as the other modes' slices."""
import numpy as np
import pytest

import gpu_util as GU
from paper_1904_03329_amd import HbcsfTensor, binding as B

pytestmark = pytest.mark.gpu


def _coo(rng, dims, nnz):
    keep = np.unique(rng.integers(0, int(np.prod(dims)), nnz))
    rng.shuffle(keep)
    return [x.astype(np.uint32) for x in np.unravel_index(keep, dims)], rng.uniform(-1, 1, keep.size).astype(np.float32)


def _on_device(inds, vals):
    import torch

    return [torch.from_numpy(x.view(np.int32)).cuda() for x in inds], torch.from_numpy(vals).cuda()


@pytest.mark.parametrize("dims,nnz", [((200, 40, 30), 40000), ((5000, 400, 60), 30000), ((60, 20, 30, 10), 50000),
                                      ((900, 300, 20, 8), 20000), ((30, 20, 10, 12, 9), 60000)])
@pytest.mark.parametrize("opts", [{}, dict(group_mask=4), dict(mid_blocking=2), dict(hybrid_granularity=1)])
def test_same_arrays_wherever_they_lie(oracle, dims, nnz, opts):
    import torch

    rng = np.random.default_rng(nnz)
    inds, vals = _coo(rng, dims, nnz)
    di, dv = _on_device(inds, vals)
    host = HbcsfTensor(dims, inds, vals, **opts)
    pieces = HbcsfTensor.from_device_coo(dims, di, dv, **opts)
    whole = HbcsfTensor.from_device_coo(dims, di, dv, compact=False, **opts)
    n = B.device_bytes(host.handle)
    assert n == B.device_bytes(pieces.handle) == B.device_bytes(whole.handle) == sum(p.numel() for p in pieces._arena)
    moved = torch.empty(n, dtype=torch.uint8, device="cuda")
    B.relocate(whole.handle, moved.data_ptr(), n, torch.cuda.current_stream().cuda_stream)
    whole._arena = moved
    facs = [rng.uniform(0, 1, (d, 16)).astype(np.float32) for d in dims]
    dev = [torch.from_numpy(f).cuda() for f in facs]
    for mode in range(len(dims)):
        want = oracle.mttkrp(dims, inds, vals, facs, mode)
        for t in (pieces, whole):
            for call in range(2):
                GU.assert_close(t.mttkrp(mode, dev).cpu().numpy(), want, f"mode {mode}, call {call}")
            a, b = dict(host.stats(mode)), dict(t.stats(mode))
            a.pop("build_seconds"), b.pop("build_seconds")
            assert a == b
    for t in (host, pieces, whole):
        t.close()


def test_memory_that_is_not_given():
    import torch

    dims = (50, 40, 30)
    inds, vals = _coo(np.random.default_rng(2), dims, 3000)
    di, dv = _on_device(inds, vals)
    ws = torch.empty(B.device_build_bytes(dims, len(vals))[1], dtype=torch.uint8, device="cuda")
    big = torch.empty(1 << 22, dtype=torch.uint8, device="cuda")

    def build(allocate):
        return B.build_format_device_pieces(dims, len(vals), [x.data_ptr() for x in di], dv.data_ptr(), allocate, ws.data_ptr(),
                                            ws.numel())

    asked = []
    for refused in range(4):   # three modes, the words of state
        asked.clear()

        def some(n):
            asked.append(n)
            return None if len(asked) == refused + 1 else big.data_ptr() + (len(asked) << 18)

        with pytest.raises(B.HbcsfError) as e:
            build(some)
        assert e.value.code == -3 and len(asked) == refused + 1
    with pytest.raises(B.HbcsfError) as e:
        build(lambda n: big.data_ptr() + 128)
    assert e.value.code == -1

    def fails(n):
        raise MemoryError("none left")

    with pytest.raises(MemoryError):
        build(fails)
    torch.cuda.synchronize()


@pytest.mark.parametrize("nnz", [39_999, 40_000, 40_001])
@pytest.mark.parametrize("dims", [(10_000, 9_000, 30), (10_000, 9_000, 40, 30)])
def test_rows_that_are_looked_up_before_they_are_marked(dims, nnz):
    """From four nonzeros per leaf row on; mode 1's leaf is the first mode.  Its three groups have row maps, and their distinct rows
    are the host builder's."""
    rng = np.random.default_rng(nnz)
    inds = np.stack([rng.integers(0, d, 2 * nnz) for d in dims])
    inds[1, ::2] %= 100   # half of it in a hundred slices, the rest thin
    flat = np.unique(np.ravel_multi_index(inds, dims))
    rng.shuffle(flat)
    inds = [x.astype(np.uint32) for x in np.unravel_index(flat[:nnz], dims)]
    vals = rng.uniform(-1, 1, nnz).astype(np.float32)
    host = HbcsfTensor(dims, inds, vals)
    assert host.stats(1)["level_mode"][len(dims) - 1] == 0 and all(host.stats(1)["group_nnz"])
    dev = HbcsfTensor.from_device_coo(dims, *_on_device(inds, vals))
    for mode in range(len(dims)):
        a, b = dict(host.stats(mode)), dict(dev.stats(mode))
        a.pop("build_seconds"), b.pop("build_seconds")
        assert a == b
    host.close()
    dev.close()
