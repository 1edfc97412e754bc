"""Calls that define the output in the launch of the group kernels: words of 32 rows at the edges of a mode's length, rows that
every block adds to, calls one after the other and from several threads, and the calls that are served with a launch of their
own instead (other streams, captured calls, long modes).  The arena ends with the modes' words of state: they say which it was."""
import threading

import numpy as np
import pytest

import gpu_util as GU
from paper_1904_03329_amd import HbcsfTensor, binding as B

pytestmark = pytest.mark.gpu


def _tensor(rng, dims, nnz, heavy):
    """Distinct coordinates; `heavy`: half of the nonzeros lie in one slice of every mode where there is room."""
    inds = np.stack([rng.integers(0, d, nnz) for d in dims])
    for m, d in enumerate(dims):
        inds[m, rng.random(nnz) < heavy] = d // 2
    keep = np.unique(np.ravel_multi_index(inds, dims))
    rng.shuffle(keep)
    inds = [x.astype(np.uint32) for x in np.unravel_index(keep, dims)]
    return inds, rng.uniform(-1, 1, keep.size).astype(np.float32)


def _state(ht, mode):
    """The words of state of a mode of `ht` (copies)."""
    import torch

    sizes = [(d + 31) // 32 * 4 for d in ht.dims]
    ends = [(n + 255) // 256 * 256 for n in sizes]
    at = ht._arena.numel() - sum(ends[mode:])
    return ht._arena[at:at + sizes[mode]].view(torch.int32).cpu().numpy().copy()


@pytest.mark.parametrize("dims,nnz,heavy,rank,dtype", [
    ((33, 32, 31), 4000, 0.0, 8, np.float32), ((1, 700, 65), 9000, 0.0, 16, np.float32), ((4000, 64, 5), 30000, 0.5, 32, np.float32),
    ((2049, 300, 40), 60000, 0.3, 64, np.float32), ((500, 97, 20), 20000, 0.5, 128, np.float32),
    ((700, 130, 33, 12), 40000, 0.4, 32, np.float32), ((300, 40, 30, 20, 9), 30000, 0.3, 16, np.float32),
    ((3001, 90, 35), 30000, 0.5, 16, np.float64), ((600, 50, 33, 7), 20000, 0.4, 64, np.float64)])
def test_rows_are_defined_once(oracle, dims, nnz, heavy, rank, dtype):
    import torch

    rng = np.random.default_rng(rank + len(dims))
    inds, vals = _tensor(rng, dims, nnz, heavy)
    facs = [rng.uniform(0, 1, (d, rank)).astype(dtype) for d in dims]
    ref, tol = (oracle.mttkrp_f64, GU.REL_TOL_F64) if dtype == np.float64 else (oracle.mttkrp, GU.REL_TOL)
    print(dims, vals.size, rank, dtype.__name__, flush=True)
    ht = HbcsfTensor(dims, inds, vals).to_device()
    dev = [torch.from_numpy(f).cuda() for f in facs]
    for mode in range(len(dims)):
        want = ref(dims, inds, vals, facs, mode)
        assert not _state(ht, mode).any()
        for call in range(1, 40):
            out = torch.full((dims[mode], rank), float("nan"), dtype=dev[0].dtype, device="cuda")
            ht.mttkrp(mode, dev, out)
            if call in (1, 2, 39):
                GU.assert_close(out.cpu().numpy(), want, f"mode {mode}, call {call}", tol)
                assert (_state(ht, mode) == 2 * call + 2).all()
            else:
                last = out
        GU.assert_close(last.cpu().numpy(), want, f"mode {mode}", tol)
    ht.close()


def test_where_the_output_is_defined_before(oracle):
    """Other streams, captured calls, profiled and tuned ones, slices in pieces, long modes: right, and without the state."""
    import torch

    rng = np.random.default_rng(5)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    dims = (512 * cus, 512 * cus + 1, 12)
    inds, vals = _tensor(rng, dims, 40000, 0.2)
    facs = [rng.uniform(0, 1, (d, 16)).astype(np.float32) for d in dims]
    want = [oracle.mttkrp(dims, inds, vals, facs, m) for m in range(3)]
    ht = HbcsfTensor(dims, inds, vals).to_device()
    dev = [torch.from_numpy(f).cuda() for f in facs]

    def check(what, mode, got, uses):
        torch.cuda.synchronize()
        GU.assert_close(got.cpu().numpy(), want[mode], what)
        now = _state(ht, mode)
        assert (now != before[mode]).all() if uses else (now == before[mode]).all(), what
        before[mode] = now

    before = [_state(ht, m) for m in range(3)]
    check("longest", 0, ht.mttkrp(0, dev), True)
    check("too long", 1, ht.mttkrp(1, dev), False)
    check("short", 2, ht.mttkrp(2, dev), True)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    out = torch.empty_like(dev[2])
    with torch.cuda.stream(side):
        check("other stream", 2, ht.mttkrp(2, dev), False)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            ht.mttkrp(2, dev, out)
    torch.cuda.current_stream().wait_stream(side)
    for _ in range(3):
        out.fill_(float("nan"))
        graph.replay()
        check("replayed", 2, out, False)
        check("short, between replays", 2, ht.mttkrp(2, dev), True)
    for key, value, back in ((B.TUNE_FUSE_COO, 0, 2), (B.TUNE_PERSISTENT, 1, 0), (B.TUNE_PROFILE, 2, 0)):
        B.tune(ht.handle, key, value)
        check(f"tuned {key}", 2, ht.mttkrp(2, dev), False)
        B.tune(ht.handle, key, back)
    check("short again", 2, ht.mttkrp(2, dev), True)
    ht.close()
    for opts in (dict(hybrid_granularity=1, fiber_threshold=8), dict(mid_blocking=2)):
        ht = HbcsfTensor(dims, inds, vals, **opts).to_device()
        before = [_state(ht, m) for m in range(3)]
        check(str(opts), 2, ht.mttkrp(2, dev), False) if "hybrid_granularity" in opts else None
        check(str(opts), 0, ht.mttkrp(0, dev), False)
        ht.close()


@pytest.mark.parametrize("rows, used, nnz, rank, uses", [   # per compute unit; a wavefront for 32 rows, of 22 there is room for
    (396, 150, 3800, 32, True), (397, 150, 3800, 32, False),          # words on 9 / 16 of them
    (512, 200, 7680, 16, True), (512, 200, 7670, 16, False),          # 15 nonzeros a row
    (512, 320, 3800, 32, True), (512, 290, 3800, 32, False),          # half of the rows stored by their slices
    (512, 200, 760, 16, True), (512, 200, 776, 16, False),            # 16 wavefronts of words, units of 128 nonzeros for the others
    (512, 200, 380, 32, True), (512, 200, 388, 32, False),            # units of 64
    (430, 200, 430, 32, True), (430, 200, 434, 32, False)])           # an output of more than 8 MiB: a nonzero a row at most
def test_long_modes(oracle, rows, used, nnz, rank, uses):
    """`used` rows have nonzeros, in pairs, so that no slice has a single one."""
    import torch

    rng = np.random.default_rng(nnz)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rows, nnz = rows * cus, nnz * cus
    dims = (rows, 60, 40)
    fiber = rng.choice(used * cus * 30, nnz // 2, replace=False)
    inds = [np.concatenate([x, x]).astype(np.uint32) for x in (fiber // 30, fiber % 30)]
    inds.append(np.repeat(np.arange(2, dtype=np.uint32), nnz // 2))
    vals = rng.uniform(-1, 1, nnz).astype(np.float32)
    facs = [rng.uniform(0, 1, (d, rank)).astype(np.float32) for d in dims]
    ht = HbcsfTensor(dims, inds, vals).to_device()
    got = ht.mttkrp(0, [torch.from_numpy(f).cuda() for f in facs])
    GU.assert_close(got.cpu().numpy(), oracle.mttkrp(dims, inds, vals, facs, 0))
    print(rows, nnz, rank, "owned", ht.stats(0)["owned_rows"], flush=True)
    assert sum(ht.stats(0)["group_nnz"][1:]) == nnz
    assert (_state(ht, 0) > 0).all() if uses else not _state(ht, 0).any()
    ht.close()


def test_threads_share_the_stream(oracle):
    """Calls of one mode from several threads on the null stream, each into its own output."""
    import torch

    rng = np.random.default_rng(6)
    dims = (900, 200, 30)
    inds, vals = _tensor(rng, dims, 50000, 0.4)
    facs = [[rng.uniform(0, 1, (d, 32)).astype(np.float32) for d in dims] for _ in range(4)]
    ht = HbcsfTensor(dims, inds, vals).to_device()
    dev = [[torch.from_numpy(f).cuda() for f in fs] for fs in facs]
    outs = [torch.full((dims[0], 32), float("nan"), device="cuda") for _ in facs]
    torch.cuda.synchronize()

    def work(k):
        for _ in range(200):
            ht.mttkrp(0, dev[k], outs[k])

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for k in range(4):
        GU.assert_close(outs[k].cpu().numpy(), oracle.mttkrp(dims, inds, vals, facs[k], 0), f"thread {k}")
    assert (_state(ht, 0) == 2 * 800 + 2).all()
    ht.close()
