"""GPU parity where a unit's parts, not only its runs, have edges: every part size the launch chooses by rank and length."""
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
    for steps in (None, 8):
        outs, _ = GU.gpu_mttkrp_all_modes(dims, t.inds, t.vals, facs, tune_steps=steps)
        for mode in range(len(dims)):
            GU.assert_close(outs[mode], want[mode], f"rank {rank} mode {mode} steps {steps}")
