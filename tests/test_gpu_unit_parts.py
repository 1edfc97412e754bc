"""GPU parity where a unit's parts, not only its runs, have edges: every part size the launch chooses by rank and length."""
import numpy as np
import pytest

import gpu_util as GU

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank", [8, 16, 32, 64, 128])
@pytest.mark.parametrize("dims, nnz, alpha", [
    ((7, 500, 900), 40_001, (0.5, 0.0, 1.0)),              # a few slices over many units, parts shorter than runs
    ((3000, 50, 40), 64 * 100 + 1, (0.0, 0.8, 0.8)),       # several slices end in one part; one nonzero beyond a unit
    ((60, 1500, 900), 1_300_000, (1.0, 1.0, 1.0)),         # units of 256 nonzeros
    ((900, 60, 30, 20), 250_000, (1.2, 1.0, 0.8, 0.0)),    # order 4: a slice list per part, fibers cut at two levels
    ((40, 30, 20, 10, 9), 63, (0.0,) * 5),                 # less than one run
])
def test_every_part_size(oracle, synth, rank, dims, nnz, alpha):
    t = synth.tensor(dims, nnz, alpha, seed=rank + len(dims))
    facs = synth.factors(dims, rank, seed=5)
    want = [oracle.mttkrp(dims, t.inds, t.vals, facs, mode) for mode in range(len(dims))]
    for steps in (None, 8) if rank == 32 else (None,):   # a choice at rows of 128 bytes only
        outs, _ = GU.gpu_mttkrp_all_modes(dims, t.inds, t.vals, facs, tune_steps=steps)
        for mode in range(len(dims)):
            GU.assert_close(outs[mode], want[mode], f"rank {rank} mode {mode} steps {steps}")


@pytest.mark.parametrize("dims, opts, run", [
    ((900, 60, 30), dict(fiber_threshold=8), 8), ((900, 60, 30), dict(fiber_threshold=16), 16),
    ((900, 60, 30), dict(fiber_threshold=32), 32), ((900, 60, 30), dict(), 64),
    ((900, 60, 30, 20), dict(), 32), ((900, 60, 30, 20), dict(fiber_threshold=64), 64),
    ((90, 60, 30, 20, 10), dict(), 32), ((90, 60, 30, 20, 10), dict(fiber_threshold=64), 64),
])
@pytest.mark.parametrize("rank, dtype", [(32, np.float32), (16, np.float64)])
def test_gathers_in_flight_setting(oracle, synth, dims, opts, run, rank, dtype):
    """HBCSF_TUNE_STEPS at rows of 128 bytes: 8 walks whole runs at every run length (a trace counts the wavefronts, one per
    unit of 8 runs on a tensor this small, in whole sets of 8 workgroups of 1, 2 or 4), 4 and 0 short parts again."""
    import torch

    from paper_1904_03329_amd import HbcsfTensor, binding as B

    t = synth.tensor(dims, 20_001, (1.0,) * len(dims), seed=9)
    facs = [f.astype(dtype) for f in synth.factors(dims, rank, seed=5)]
    ref, tol = (oracle.mttkrp_f64, GU.REL_TOL_F64) if dtype == np.float64 else (oracle.mttkrp, GU.REL_TOL)
    want = [ref(dims, t.inds, t.vals, facs, mode) for mode in range(len(dims))]
    ht = HbcsfTensor(dims, t.inds, t.vals, group_mask=4, **opts).to_device()
    buf = torch.zeros(4 + 4 * 8192, dtype=torch.int64, device="cuda")
    B.tune(ht.handle, B.TUNE_TRACE_CAPACITY, 8192)
    B.tune(ht.handle, B.TUNE_TRACE_BUFFER, buf.data_ptr())
    dfacs = [torch.from_numpy(f).cuda() for f in facs]
    waves = {}
    for steps in (4, 8, 0):
        B.tune(ht.handle, B.TUNE_STEPS, steps)
        for mode in range(len(dims)):
            buf.zero_()
            out = ht.mttkrp(mode, dfacs).cpu().numpy()
            waves[steps] = int(buf[0])
            GU.assert_close(out, want[mode], f"{dims} {opts} steps {steps} mode {mode}", tol)
    units = -(-len(t.vals) // (8 * run))
    assert waves[8] in [-(-units // (8 * w)) * 8 * w for w in (1, 2, 4)]
    assert waves[0] == waves[4] and (waves[4] > waves[8] if run > 8 else waves[4] == waves[8])
    ht.close()


@pytest.mark.parametrize("dims, opts", [((900, 60, 30), dict()), ((900, 60, 30, 20), dict())])
@pytest.mark.parametrize("steps", [0, 4, 8])
def test_dense_gather_with_each_setting(oracle, synth, dims, opts, steps):
    t = synth.tensor(dims, 20_001, (1.0,) * len(dims), seed=9)
    facs = synth.factors(dims, 32, seed=5)
    outs, _ = GU.gpu_mttkrp_all_modes(dims, t.inds, t.vals, facs, tune_dense=1, tune_steps=steps, group_mask=4, **opts)
    for mode, out in enumerate(outs):
        GU.assert_close(out, oracle.mttkrp(dims, t.inds, t.vals, facs, mode), f"{dims} steps {steps} mode {mode}")
