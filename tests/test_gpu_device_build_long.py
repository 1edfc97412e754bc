"""Device builds on both sides of 2^30 nonzeros, from which on the pairs of 64-bit keys are sorted by rocPRIM: plain, with a blocked
order (two sorts a mode there) and with the per-fiber choice.  Values and factors are small integers, so that every sum is exact in
double precision (at most 2^30 terms of magnitude 12, below 2^53) and the results have to be equal."""
import pytest

pytestmark = pytest.mark.gpu

DIMS = (2003, 3001, 5003)


@pytest.mark.parametrize("nnz, opts", [(2**30 - 1, {}), (2**30 - 1, dict(mid_blocking=4)), (2**30, {}), (2**30, dict(mid_blocking=4)),
                                       (2**30, dict(hybrid_granularity=1))])
def test_both_sorts(nnz, opts):
    import torch
    from paper_1904_03329_amd import HbcsfTensor

    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 160 << 30:
        pytest.skip("needs 160 GB of device memory")
    print(nnz, opts, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(nnz % 1000)
    inds = [torch.randint(0, d, (nnz,), generator=gen, device="cuda", dtype=torch.int32) for d in DIMS]
    vals = torch.randint(-3, 4, (nnz,), generator=gen, device="cuda", dtype=torch.int8).float()
    facs = [torch.randint(-2, 3, (d, 16), generator=gen, device="cuda").double() for d in DIMS]
    ht = HbcsfTensor.from_device_coo(DIMS, inds, vals, **opts)
    print("built", flush=True)
    for mode in range(3):
        assert ht.stats(mode)["slices"] >= DIMS[mode] and sum(ht.stats(mode)["group_nnz"]) == nnz
        got = ht.mttkrp(mode, facs)
        others = [m for m in range(3) if m != mode]
        for column in (0, 15):
            want = torch.zeros(DIMS[mode], dtype=torch.float64, device="cuda")
            for part in range(0, nnz, 1 << 27):
                s = slice(part, min(part + (1 << 27), nnz))
                terms = vals[s].double()
                for m in others:
                    terms *= facs[m][:, column].contiguous().index_select(0, inds[m][s])
                want += torch.bincount(inds[mode][s], weights=terms, minlength=DIMS[mode])
                del terms
            assert torch.equal(got[:, column], want), (mode, column)
        print("mode", mode, "equal", flush=True)
    ht.close()
    del ht, inds, vals
    torch.cuda.empty_cache()
