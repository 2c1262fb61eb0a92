"""The work that a program using this library has it do, as cases that can be timed and compared.

Shapes are those of the library's own workloads (``workloads.py``: a single linear, feed-forward pairs and
transformer layers with hidden sizes 1024 to 8192) and of its serving entry point, plus the ragged sizes that real
batches bring: token counts are whatever a batch holds, and slices are as wide as the granularity leaves them.

A case is one of
  step     forward of every operator, then backward in reverse order: one training pass over the operators of a
           layer, with a compute and a copy stream and one workspace for all of them;
  forward  one operator's forward on one stream with the library's built-in scratch memory (serving);
  gather   one column slice pulled together from the shards.
Everything is bf16 with fp32 sums, the only type the library takes.
"""
from __future__ import annotations

import math
from typing import Dict, List, Tuple

import torch

import paper_2209_13258_amd as osdp

STAGING = {"auto": osdp.OSDP_STAGING_AUTO, "single": osdp.OSDP_STAGING_SINGLE, "double": osdp.OSDP_STAGING_DOUBLE,
           "half": osdp.OSDP_STAGING_HALF}
SPLIT = {"out": osdp.OSDP_SPLIT_OUT_FEATURES, "in": osdp.OSDP_SPLIT_IN_FEATURES, "longer": osdp.OSDP_SPLIT_LONGER,
         "per_pass": osdp.OSDP_SPLIT_PER_PASS}
# name of the layout -> its operators as (in-features, out-features) in units of the hidden size and the inner size
LAYOUTS = {
    "linear": lambda h, f: [(h, f)],
    "ffn": lambda h, f: [(h, f), (f, h)],
    "layer": lambda h, f: [(h, 3 * h), (h, h), (h, f), (f, h)],
}
DRAWN_FLOPS = 2.0e12  # a drawn case stays far below the largest listed one (1.3e13) even on a path five times slower


def _step(name: str, layout: str, T: int, h: int, f: int, k: str, N: int = 8, split: str = "out", staging: str = "auto",
          zdp_of_8: int = 8) -> Dict:
    return {"name": name, "kind": "step", "layout": layout, "T": T, "h": h, "f": f, "k": k, "N": N, "split": split,
            "staging": staging, "zdp_of_8": zdp_of_8}


def listed() -> List[Dict]:
    return [
        # the smallest training call: latency and launches
        _step("linear-t128-256x1024", "linear", 128, 256, 1024, "4", N=2),
        # serving, one token of one sequence: the weights are read for a single row
        {"name": "serve-t1-4096x16384", "kind": "forward", "T": 1, "h": 4096, "f": 16384, "k": "8", "N": 8},
        # serving, a batch of sequences: still far fewer rows than a matrix-core tile of the large kernels
        {"name": "serve-t33-8192x32768", "kind": "forward", "T": 33, "h": 8192, "f": 32768, "k": "8", "N": 8},
        # serving, a prompt of a few hundred tokens that no tile divides
        {"name": "prompt-t500-2560x10240", "kind": "forward", "T": 500, "h": 2560, "f": 10240, "k": "4", "N": 8},
        # feed-forward pair of a small model, large batch
        _step("ffn-h1024-t8192", "ffn", 8192, 1024, 4096, "4,4"),
        # a whole layer with a per-operator granularity
        _step("layer-h2560-t16384", "layer", 16384, 2560, 10240, "2,1,4,4"),
        # wide operators, where splitting is what bounds the memory
        _step("wide-ffn-h8192-t4096", "ffn", 4096, 8192, 32768, "8,8"),
        # one layer of a larger model, with the seeded plan of its workload
        _step("layer-h4096-t8192", "layer", 8192, 4096, 16384, "2,4,4,4"),
        # a layer over a batch packed from sequences of different lengths: an odd number of tokens
        _step("packed-layer-h2560-t3001", "layer", 3001, 2560, 10240, "2,1,4,4"),
        # the finest granularity the library proposes by default: slices of 640 and 160 columns
        _step("fine-slices-h2560-t8192", "ffn", 8192, 2560, 10240, "16,16"),
        # half of the slices replicated, half sharded, each operator cut along its longer dimension
        _step("half-zdp-ffn-h4096-t2048", "ffn", 2048, 4096, 16384, "8,8", split="longer", zdp_of_8=4),
        # a slice gathered by itself, ahead of its use
        {"name": "gather-8192x32768-k8", "kind": "gather", "T": 1, "h": 8192, "f": 32768, "k": "8", "N": 8},
    ]


def _log_int(rng, lo: int, hi: int) -> int:
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _width(rng, lo: int, hi: int, unit: int) -> int:
    """A feature count over [lo, hi]: mostly what models have (multiples of 256 and 64), now and then any multiple of
    8; always a multiple of ``unit``, so that every slice starts on 8 features."""
    step = rng.choice([256, 256, 64, 8])
    step = step * unit // math.gcd(step, unit)
    return max(1, round(_log_int(rng, lo, hi) / step)) * step


def draw(rng) -> Dict:
    while True:
        kind = rng.choice(["step", "step", "step", "forward", "forward", "gather"])
        k = rng.choice([1, 2, 3, 4, 6, 8, 16])
        N = rng.choice([1, 2, 4, 8, 8])
        unit = 16 * k
        h, f = _width(rng, 256, 8192, unit), _width(rng, 512, 32768, unit)
        case = {"kind": kind, "h": h, "f": f, "N": N}
        if kind == "step":
            layout = rng.choice(["linear", "ffn", "layer"])
            T = _log_int(rng, 64, 16384)
            if rng.random() < 0.5:  # half of the batches are padded to a whole number of tiles
                T = (T + 127) // 128 * 128
            split = rng.choice(["out", "out", "in", "longer", "per_pass"])
            staging = rng.choice(["auto", "auto", "auto", "single", "double", "half"])
            zdp = rng.choice([8, 8, 8, 4, 1]) if split != "per_pass" and k > 1 else 8
            case.update(layout=layout, T=T, k=",".join([str(k)] * len(LAYOUTS[layout](h, f))), split=split, staging=staging,
                        zdp_of_8=zdp)
        elif kind == "forward":
            case.update(T=_log_int(rng, 1, 512), k=str(k))
            if h * (f // k) * 2 > osdp.OSDP_NOALLOC_SCRATCH_BYTES // 2:
                continue
        else:
            case.update(T=1, k=str(k))
        if kind == "gather" and h * (f // k) < 1 << 14:
            continue
        if work(case)["flops"] <= DRAWN_FLOPS and work(case)["bytes"] <= 4e9:
            return case


def _operators(case) -> List[Tuple[int, int]]:
    layout = case["layout"] if case["kind"] == "step" else "linear"
    return LAYOUTS[layout](case["h"], case["f"])


def _granularities(case) -> List[int]:
    return [int(v) for v in case["k"].split(",")]


def _normal(shape, gen, std: float = 1.0) -> torch.Tensor:
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(std).to(torch.bfloat16)


def _weights(I: int, O: int, N: int, gen) -> List[torch.Tensor]:
    return [_normal(((I * O + N - 1) // N,), gen, 0.02) for _ in range(N)]


def prepare(case, seed: int):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    T, N = case["T"], case["N"]
    ops, ks = _operators(case), _granularities(case)
    st = {"case": case, "ks": ks, "ops": []}
    if case["kind"] == "gather":
        (I, O), k = ops[0], ks[0]
        st["slice"] = seed % k
        st["W"] = _weights(I, O, N, gen)
        st["staging"] = torch.empty((I, O // k), device="cuda", dtype=torch.bfloat16)
        return st
    for I, O in ops:
        op = {"X": _normal((T, I), gen), "W": _weights(I, O, N, gen),
              "Y": torch.empty((T, O), device="cuda", dtype=torch.bfloat16)}
        if case["kind"] == "step":
            op["dY"] = _normal((T, O), gen)
            op["dX"] = torch.empty((T, I), device="cuda", dtype=torch.bfloat16)
            op["dW"] = [torch.empty_like(w) for w in op["W"]]
        st["ops"].append(op)
    if case["kind"] == "forward":
        return st

    plan = osdp.Plan(ks, staging=STAGING[case["staging"]], split_dim_per_op=[SPLIT[case["split"]]] * len(ops))
    st["mixed"] = case["zdp_of_8"] < 8
    if st["mixed"]:  # the first slices stay sharded, the others are read from a resident replica of the matrix
        plan.zdp_mask = []
        for (I, O), k, op in zip(ops, ks, st["ops"]):
            z = max(1, k * case["zdp_of_8"] // 8)
            rows = case["split"] == "in" or (case["split"] == "longer" and I > O)
            full, dfull = _normal((I, O), gen, 0.02), torch.zeros((I, O), device="cuda", dtype=torch.bfloat16)
            for w in op["dW"]:
                w.zero_()  # the replicated slices' part of the sharded gradient is never written
            starts = [(j * I // k) * O if rows else j * O // k for j in range(k)]
            op["w_dp"] = [None if j < z else full.view(-1)[s:] for j, s in enumerate(starts)]
            op["dw_dp"] = [None if j < z else dfull.view(-1)[s:] for j, s in enumerate(starts)]
            op["ld_dp"], op["dW_dp"] = O, dfull
            plan.zdp_mask.append((1 << z) - 1)
    need = 256
    for n, ((I, O), k) in enumerate(zip(ops, ks)):
        for is_bwd in (False, True):
            need = max(need, osdp.osdp_split_linear_workspace_bytes(T, I, O, N, k, is_bwd, plan, n)[0])
    st["plan"] = plan
    st["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    st["copy"] = torch.cuda.Stream()
    return st


def run(st):
    case = st["case"]
    compute = torch.cuda.current_stream()
    if case["kind"] == "gather":
        osdp.osdp_split_linear_gather_slice(case["h"], case["f"], st["ks"][0], st["slice"], st["W"], st["staging"], compute)
        return st["staging"]
    if case["kind"] == "forward":
        op = st["ops"][0]
        osdp.osdp_split_linear_fwd_noalloc(op["X"], op["W"], op["Y"], st["ks"][0], stream=compute)
        return op["Y"]
    opts = dict(plan=st["plan"], stream_compute=compute, stream_copy=st["copy"])
    ops = list(enumerate(zip(st["ops"], st["ks"])))
    for n, (op, k) in ops:
        if st["mixed"]:
            osdp.osdp_split_linear_fwd_mixed(op["X"], op["W"], op["w_dp"], op["ld_dp"], op["Y"], k, st["ws"], op_index=n, **opts)
        else:
            osdp.osdp_split_linear_fwd(op["X"], op["W"], op["Y"], k, st["ws"], op_index=n, **opts)
    for n, (op, k) in reversed(ops):
        if st["mixed"]:
            osdp.osdp_split_linear_bwd_mixed(op["X"], op["dY"], op["W"], op["w_dp"], op["ld_dp"], op["dX"], op["dW"],
                                             op["dw_dp"], k, st["ws"], op_index=n, **opts)
        else:
            osdp.osdp_split_linear_bwd(op["X"], op["dY"], op["W"], op["dX"], op["dW"], k, st["ws"], op_index=n, **opts)
    outs = ("Y", "dX", "dW", "dW_dp") if st["mixed"] else ("Y", "dX", "dW")
    return [{name: op[name] for name in outs} for op in st["ops"]]


def work(case) -> Dict[str, float]:
    T = case["T"]
    total = {"bytes": 0.0, "flops": 0.0}
    for (I, O), k in zip(_operators(case), _granularities(case)):
        if case["kind"] == "gather":
            total["bytes"] += 2 * 2.0 * I * (O // k)
        elif case["kind"] == "forward":
            total["bytes"] += 2.0 * (T * I + I * O + T * O)
            total["flops"] += 2.0 * T * I * O
        else:  # X, dY and W in; Y, dX and dW out
            total["bytes"] += 2.0 * (2 * T * I + 2 * T * O + 2 * I * O)
            total["flops"] += 6.0 * T * I * O
    return total


def tolerance(case):
    if case["kind"] == "gather":
        return "exact"
    # one bf16 rounding of an fp32 sum: against the same product in 64 bits the results differ by 1.7e-3 in the
    # 2-norm and by at most 2^-8 of a value (half a step just above a power of two); four times that
    return {"rel": 7e-3, "max": 1.6e-2}
