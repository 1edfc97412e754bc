"""The work users of this framework have it do, as timed cases: MTTKRP over all modes of a resident tensor, CPD-ALS
decompositions, and the way from a new COO tensor (device or host memory) to its first MTTKRP results.

`listed` are fixed cases, `draw` gives further ones of the same ranges.  A case is a dict:
    kind     "mttkrp": MTTKRP of every mode on a resident tensor;  "als": a CPD-ALS decomposition on one;
             "device": format build from COO arrays on the GPU, then MTTKRP of every mode;
             "host": format build from COO arrays in host memory, upload, then MTTKRP of every mode
    dims, alpha   texts, one entry per mode: dimension and Zipf exponent of the index law (0 = uniform)
    nnz, rank, dtype ("f32" / "f64": factors, sums and results; a tensor's values are always float32)
    iterations    ALS iterations ("als" only)
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1904_03329_amd import CpdAls, HbcsfTensor


def _case(kind, dims, nnz, alpha, rank, dtype="f32", iterations=0, name=None):
    c = {} if name is None else {"name": name}
    c.update(kind=kind, dims="x".join(str(d) for d in dims), nnz=int(nnz), alpha=",".join(str(a) for a in alpha),
             rank=int(rank), dtype=dtype, iterations=int(iterations))
    return c


def listed():
    return [
        # The benchmark's five configurations: a tiny tensor whose calls are all latency, ...
        _case("mttkrp", (100, 80, 60), 10_000, (0, 0, 0), 8, name="cfg1"),
        # ... (a small skewed one, as in interactive use and the smoke test) ...
        _case("mttkrp", (3000, 400, 60), 80_000, (1.3, 1.1, 1.0), 32, name="small"),
        # ... a medium power-law tensor, ...
        _case("mttkrp", (100_000, 100_000, 10_000), 5_000_000, (1.2, 1.2, 1.2), 32, name="cfg2"),
        # ... one with extreme slice skew, whose factor matrices stay in the caches, ...
        _case("mttkrp", (480_000, 18_000, 2_000), 100_000_000, (1.5, 1.1, 1.1), 32, name="cfg3"),
        # ... an order-4 one, ...
        _case("mttkrp", (1_000_000, 50_000, 5_000, 1_000), 50_000_000, (1.3, 1.1, 1.0, 0.8), 32, name="cfg4"),
        # ... and the hypersparse long-tail one, whose factor matrices and outputs are 5 GB each.
        _case("mttkrp", (40_000_000, 40_000_000, 1_000), 150_000_000, (1.05, 1.05, 0), 32, name="cfg5"),
        # The shape of a noun-verb-noun tensor (12K x 9K x 29K) at a tenth of its nonzeros, odd sizes, a lower rank.
        _case("mttkrp", (12_101, 9_187, 28_819), 7_700_001, (1.1, 1.1, 1.0), 16, name="ragged_r16"),
        # Double precision factors and results.
        _case("mttkrp", (100_000, 100_000, 10_000), 5_000_000, (1.2, 1.2, 1.2), 32, dtype="f64", name="cfg2_f64"),
        # Decompositions: the medium tensor at the usual rank, and a smaller one at a higher rank.
        _case("als", (100_000, 100_000, 10_000), 5_000_000, (1.2, 1.2, 1.2), 32, iterations=5, name="als_cfg2"),
        _case("als", (30_011, 4_003, 601), 801_003, (1.3, 1.1, 1.0), 64, iterations=5, name="als_r64"),
        # A new tensor that is already in device memory: order 4, built on the GPU and used once per mode.
        _case("device", (1_000_000, 50_000, 5_000, 1_000), 50_000_000, (1.3, 1.1, 1.0, 0.8), 32, name="device_cfg4"),
        # A new tensor in host memory (numpy): host build, upload, used once per mode.
        _case("host", (100_000, 100_000, 10_000), 1_000_000, (1.2, 1.2, 1.2), 32, name="host_1m"),
    ]


# nonzeros of a drawn case, by kind (log-uniform); every one costs less than the largest listed case
_NNZ = {"mttkrp": (5_000, 80_000_000), "als": (10_000, 10_000_000), "device": (50_000, 40_000_000), "host": (20_000, 800_000)}


def draw(rng):
    kind = rng.choice(["mttkrp"] * 6 + ["als"] * 2 + ["device"] + ["host"])
    order = rng.choice([3, 3, 3, 4, 4, 5])
    lo, hi = _NNZ[kind]
    nnz = int(math.exp(rng.uniform(math.log(lo), math.log(hi)))) | 1
    dtype = "f64" if kind == "mttkrp" and rng.random() < 0.15 else "f32"
    rank = rng.choice([16, 32, 32, 64] if dtype == "f64" else [8, 16, 32, 32, 64] if kind == "als" else [8, 16, 32, 32, 32, 64, 128])
    if rank > 32:
        nnz = max(lo, nnz * 32 // rank) | 1
    while True:
        # a long mode now and then (hypersparse tensors), the others between tens and a million; few modes in use are
        # longer than the tensor has nonzeros
        dims = []
        for m in range(order):
            top = 8_000_000 if m < 2 and rng.random() < 0.2 else 1_000_000
            dims.append(int(math.exp(rng.uniform(math.log(40 if m else 300), math.log(min(top, nnz))))) | 1)
        bits = sum(math.log2(d) for d in dims)
        # sparse, packable into 63 bits, and no larger than the largest listed factors
        if math.log2(nnz) + 5 < bits < 62 and sum(dims) * rank < 80_000_000 * 8:
            break
    alpha = [rng.choice([0, 0.8, 1.0, 1.05, 1.1, 1.2, 1.3]) for _ in range(order)]
    return _case(kind, dims, nnz, alpha, rank, dtype, rng.randint(3, 8) if kind == "als" else 0)


def _shape(case):
    return [int(d) for d in case["dims"].split("x")], [float(a) for a in case["alpha"].split(",")]


def _coordinates(dims, alpha, nnz, gen):
    """Distinct coordinates in random order, one int32 tensor per mode: each index follows a bounded Zipf law (or a
    uniform one) over a random permutation of its range.  Fewer than nnz where the laws hardly reach that many."""
    laws = []
    for d, a in zip(dims, alpha):
        if a > 0:
            # weights in fixed point: a sum of integers is the same on every run, whatever the order of the scan
            cdf = torch.arange(1, d + 1, dtype=torch.float64, device="cuda").pow_(-a).mul_(2.0 ** 52).long().cumsum_(0)
            laws.append((cdf, torch.randperm(d, generator=gen, device="cuda", dtype=torch.int32)))
        else:
            laws.append(None)
    keys = torch.empty(0, dtype=torch.int64, device="cuda")
    for _ in range(10):
        new = torch.zeros(nnz + nnz // 8 + 16, dtype=torch.int64, device="cuda")
        for d, law in zip(dims, laws):
            u = torch.rand(new.shape[0], dtype=torch.float64, device="cuda", generator=gen)
            if law is None:
                i = u.mul_(d).long().clamp_(max=d - 1)
            else:
                u = u.mul_(law[0][-1].item()).long()
                i = law[1][torch.searchsorted(law[0], u, right=True, out_int32=True).clamp_(max=d - 1)]
            new.mul_(d).add_(i)
            del u, i
        keys = torch.unique(torch.cat([keys, new]))
        del new
        if keys.shape[0] >= nnz:
            break
    keys = keys[torch.randperm(keys.shape[0], generator=gen, device="cuda")[:nnz]]
    inds = []
    for d in reversed(dims):
        inds.append(torch.remainder(keys, d).int())
        keys = torch.div(keys, d, rounding_mode="floor")
    return inds[::-1]


def prepare(case, seed):
    dims, alpha = _shape(case)
    rank, kind = case["rank"], case["kind"]
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    inds = _coordinates(dims, alpha, case["nnz"], gen)
    vals = torch.rand(inds[0].shape[0], device="cuda", generator=gen).mul_(2).sub_(1)
    dtype = torch.float64 if case["dtype"] == "f64" else torch.float32
    factors = [torch.rand((d, rank), dtype=dtype, device="cuda", generator=gen) for d in dims]
    state = {"kind": kind, "dims": dims, "factors": factors}
    if kind == "host":
        state["inds"] = [i.cpu().numpy().view(np.uint32) for i in inds]
        state["vals"] = vals.cpu().numpy()
    elif kind == "device":
        state["inds"], state["vals"] = inds, vals
    else:
        state["tensor"] = HbcsfTensor.from_device_coo(dims, inds, vals)
    if kind == "als":
        # a decomposition starts from factors of both signs and is called with the program's own copies of them
        state["factors"] = [f.mul_(2).sub_(1) for f in factors]
        state["work"] = [torch.empty_like(f) for f in factors]
        state["als"] = CpdAls(state["tensor"], rank)
        state["iterations"] = case["iterations"]
    elif kind == "mttkrp":
        state["out"] = [torch.empty_like(f) for f in factors]
    torch.cuda.empty_cache()
    return state


def run(state):
    kind, factors = state["kind"], state["factors"]
    if kind == "als":
        work = state["work"]
        for w, f in zip(work, factors):
            w.copy_(f)
        done, fit = state["als"].run(work, max_iterations=state["iterations"], tolerance=0.0)
        return {"factors": work, "lambda": state["als"].lam, "done": done, "fit": fit}
    if kind == "device":
        tensor = HbcsfTensor.from_device_coo(state["dims"], state["inds"], state["vals"])
    elif kind == "host":
        tensor = HbcsfTensor(state["dims"], state["inds"], state["vals"]).to_device()
    else:
        tensor = state["tensor"]
    out = state.get("out")
    return [tensor.mttkrp(mode, factors, None if out is None else out[mode]) for mode in range(len(factors))]


def work(case):
    """Per mode: each nonzero's value and leaf index once, the other factors' reachable rows once, the result once;
    order x rank multiply-adds counted as the benchmark does (order * rank * nnz).  A build also reads the COO arrays
    and writes each mode's values and leaf indices; a decomposition also reads and writes every factor."""
    dims, _ = _shape(case)
    nnz, rank, order = case["nnz"], case["rank"], len(dims)
    elem = 8 if case["dtype"] == "f64" else 4
    rows = [min(d, nnz) * rank * elem for d in dims]
    full = [d * rank * elem for d in dims]
    nbytes = sum(8 * nnz + sum(rows) - rows[m] + full[m] for m in range(order))
    flops = order * order * rank * nnz
    if case["kind"] == "als":
        # the product with the R x R matrix and the Gram matrix of the result
        nbytes, flops = nbytes + sum(full), flops + sum(4 * d * rank * rank for d in dims)
        nbytes, flops = nbytes * case["iterations"], flops * case["iterations"]
    elif case["kind"] in ("device", "host"):
        nbytes += 4 * (order + 1) * nnz + order * 8 * nnz
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] == "als":
        # single-precision sums, amplified by the condition of the normal equations over several iterations
        return {"rel": 1e-4, "max": 4e-3}
    if case["dtype"] == "f64":
        return {"rel": 1e-12, "max": 1e-10}
    return {"rel": 1e-5, "max": 1e-3}
