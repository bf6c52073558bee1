"""The work that a user of the layer solver has it do, as cases that can be timed and compared.

A case is a dict of plain values.  `kind` names what the user's program calls:

  layer      the whole path of one layer from its calibration inputs: Hessian, inverse, pruning with
             its trace, global step, weights of the chosen mask
  calibrate  the front half alone: inputs in `batches` pieces accumulated into the dampened Hessian,
             then its inverse -- done once per layer, before any number of compressions
  refit      the front half of the sequential variant: Hessian, cross moment, re-fitted dense weights
             and the inverse
  prune      Algorithm 1 on a layer whose inverse Hessian is at hand: unstructured (all steps, then the
             global step and the weights of the mask, from the trace or by the closed form), or N:M
  blocks     the same with blocks of four weights
  quantize   min-max grid and Algorithm 3
  compound   prune to a sparsity, then quantize the survivors

The row solvers start from an inverse Hessian made here in fp64, so that what they are given depends on
the seed alone; the front half has cases of its own.
"""
import math

import torch

import paper_2208_11580_amd as obc

DEV = "cuda:0"


def listed():
    return [
        # the smallest layer of the repository's workloads, end to end: launches and waits are all it costs
        {"name": "layer_16x32", "kind": "layer", "rows": 16, "cols": 32, "samples": 256, "data": "relu",
         "sparsity": 0.5},
        # calibration of a 3x3 convolution on 64 channels (d = 576) over 50 000 patches
        {"name": "calibrate_576", "kind": "calibrate", "cols": 576, "samples": 50000, "batches": 1, "data": "relu"},
        # calibration of a 3x3 convolution on 256 channels (d = 2304): the inputs arrive in four batches
        {"name": "calibrate_2304", "kind": "calibrate", "cols": 2304, "samples": 50000, "batches": 4, "data": "relu"},
        # sequential variant on the same layer, 256 output channels
        {"name": "refit_256x2304", "kind": "refit", "rows": 256, "cols": 2304, "samples": 50000, "data": "relu"},
        # 2:4 sparsity of the 64-channel convolution: fewer rows than compute units
        {"name": "prune24_64x576", "kind": "prune", "rows": 64, "cols": 576, "data": "relu", "n": 2, "m": 4},
        # a ragged layer (odd channel counts, a bias column): no multiple of a tile anywhere, a fine
        # symmetric grid, the outlier rule
        {"name": "quant8_203x1283", "kind": "quantize", "rows": 203, "cols": 1283, "data": "relu", "bits": 8,
         "symmetric": True, "outliers": True},
        # attention projection of a BERT-base sized transformer pruned to 50 % with its trace
        {"name": "prune50_768x768", "kind": "prune", "rows": 768, "cols": 768, "data": "norm", "sparsity": 0.5,
         "recover": "trace"},
        # the first linear layer of its feed-forward block, 4 bit: many rows of moderate width
        {"name": "quant4_3072x768", "kind": "quantize", "rows": 3072, "cols": 768, "data": "norm", "bits": 4,
         "symmetric": False, "outliers": False},
        # the 256-channel 3x3 convolution, 4 bit: the benchmark's headline layer
        {"name": "quant4_256x2304", "kind": "quantize", "rows": 256, "cols": 2304, "data": "relu", "bits": 4,
         "symmetric": False, "outliers": False},
        # the same layer pruned in blocks of four
        {"name": "blocks50_256x2304", "kind": "blocks", "rows": 256, "cols": 2304, "data": "relu", "sparsity": 0.5},
        # the second linear layer of the feed-forward block, pruned; its trace would be 29 GB, so the
        # weights of the mask come from the closed form
        {"name": "prune50_768x3072", "kind": "prune", "rows": 768, "cols": 3072, "data": "norm", "sparsity": 0.5,
         "recover": "closed"},
        # the widest layers (3x3 convolution on 512 channels), one GPU's half of the rows: prune to 50 %,
        # then 4 bit on the survivors
        {"name": "compound_256x4608", "kind": "compound", "rows": 256, "cols": 4608, "data": "relu",
         "sparsity": 0.5, "bits": 4},
    ]


# the largest listed row-solver case: bounds on what draw() may give
_MOST_MATRIX = 256 * 4608 ** 2         # entries of the rows' private inverses
_MOST_STEPS = 256 * 4608 ** 3          # rows x cols^3
_MOST_TRACE = 1.9e9                    # entries of a pruning trace


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "calibrate", "refit", "prune", "prune", "blocks", "quantize", "quantize", "quantize",
                       "compound"])
    data = rng.choice(["relu", "norm"])
    if kind in ("calibrate", "refit"):
        cols = _log_int(rng, 64, 2304)
        case = {"kind": kind, "cols": cols, "samples": _log_int(rng, max(1024, 2 * cols), 50000), "data": data}
        if kind == "calibrate":
            case["batches"] = rng.choice([1, 1, 2, 4])
        else:
            case["rows"] = _log_int(rng, 16, 256)
        return case
    if kind == "layer":
        cols = _log_int(rng, 24, 64)
        return {"kind": kind, "rows": _log_int(rng, 8, 64), "cols": cols, "samples": _log_int(rng, 4 * cols, 1024),
                "data": "relu", "sparsity": round(rng.uniform(0.3, 0.8), 2)}
    cols = _log_int(rng, 48, 4608)
    if kind == "blocks":
        cols = (cols + 3) // 4 * 4
    most = min(3072, _MOST_MATRIX // 2 // cols ** 2, _MOST_STEPS // 2 // cols ** 3)
    # (quantization is chaotic: a near-tie decided the other way sends the rest of its row another way, see
    # tolerance(), so its layers have enough rows for one row to be a small share)
    least = 12 if kind in ("prune", "blocks") else 64 if cols < 512 else 200
    rows = _log_int(rng, least, max(least + 1, most))
    case = {"kind": kind, "rows": rows, "cols": cols, "data": data}
    if kind == "quantize":
        case.update(bits=rng.choice([4, 6, 8]), symmetric=rng.random() < 0.3, outliers=rng.random() < 0.3)
    elif kind == "compound":
        case.update(sparsity=round(rng.uniform(0.4, 0.7), 2), bits=rng.choice([4, 8]))
    elif kind == "blocks":
        case.update(sparsity=round(rng.uniform(0.3, 0.7), 2))
        case["rows"] = max(12, min(rows, int(4 * _MOST_TRACE / cols ** 2)))
    elif rng.random() < 0.3:
        n, m = rng.choice([(2, 4), (4, 8)])
        case.update(cols=(cols + 7) // 8 * 8, n=n, m=m)
    else:
        case.update(sparsity=round(rng.uniform(0.3, 0.8), 2),
                    recover="trace" if rows * cols ** 2 <= _MOST_TRACE else "closed")
    return case


# ------------------------------------------------------------------------------------------- inputs
def _inputs(case, gen, samples):
    """Layer inputs, d x samples fp32: correlated post-ReLU activations, or standardised tokens with a
    few heavy channels."""
    d = case["cols"]
    Z = torch.randn(d, samples, generator=gen, device=DEV)
    if case["data"] == "relu":
        A = torch.randn(d, d, generator=gen, device=DEV) / math.sqrt(d)
        A *= torch.logspace(0.0, -3.0, d, device=DEV)
        return torch.clamp_min(A @ Z, 0.0)
    X = (Z - Z.mean(dim=0, keepdim=True)) / Z.std(dim=0, unbiased=False, keepdim=True)
    heavy = torch.randperm(d, generator=gen, device=DEV)[:max(1, round(0.01 * d))]
    X[heavy] *= 10.0
    return X


def _inverse_hessian(case, gen):
    """What calibration leaves behind, fp64 inside: (2 X X^T + 1 % of its mean diagonal)^-1 as fp32."""
    d = case["cols"]
    X = _inputs(case, gen, max(256, 2 * d)).double()
    H = 2.0 * (X @ X.T)
    H.diagonal().add_(0.01 * H.diagonal().mean())
    inv = torch.cholesky_inverse(torch.linalg.cholesky(H))
    return (0.5 * (inv + inv.T)).float().contiguous()


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    kind, d = case["kind"], case["cols"]
    R = case.get("rows", 0)
    ctx = obc.Context()
    s = {"case": case, "ctx": ctx}
    if R:
        s["W"] = torch.randn(R, d, generator=gen, device=DEV) * 0.03
    if kind in ("layer", "calibrate", "refit"):
        X = _inputs(case, gen, case["samples"])
        s["H"] = torch.empty(d, d, device=DEV)
        if kind == "refit":
            # the dense layer's outputs on the dense inputs; the inputs of the partly compressed model differ
            s["Y"] = s["W"] @ X
            s["C"] = torch.empty(R, d, device=DEV)
            s["Wfit"] = torch.empty(R, d, device=DEV)
            X = X + 0.1 * X.std() * torch.randn(X.shape, generator=gen, device=DEV)
        n = case.get("batches", 1)
        edges = [case["samples"] * b // n for b in range(n + 1)]
        s["X"] = [X[:, a:b].contiguous() for a, b in zip(edges, edges[1:])]
    else:
        s["Hinv"] = _inverse_hessian(case, gen)
    if kind in ("layer", "prune", "compound", "quantize"):
        steps = d // case["m"] * (case["m"] - case["n"]) if case.get("m") else d
        s["steps"] = steps
        s["out"] = {"order": torch.full((R, steps), -1, dtype=torch.int32, device=DEV),
                    "loss": torch.zeros(R, steps, device=DEV), "W": torch.empty(R, d, device=DEV)}
        if kind == "layer" or case.get("recover") == "trace":
            s["out"]["trace"] = torch.empty(R, steps, d, device=DEV)
        if kind == "quantize":
            s["out"]["codes"] = torch.empty(R, d, dtype=torch.int32, device=DEV)
        if kind == "compound":
            s["quant"] = {"order": torch.full((R, d), -1, dtype=torch.int32, device=DEV),
                          "loss": torch.zeros(R, d, device=DEV), "W": torch.empty(R, d, device=DEV),
                          "codes": torch.empty(R, d, dtype=torch.int32, device=DEV)}
    if R and kind != "refit":
        ctx.workspace(max(ctx.rows_workspace_bytes(R, d), 1 << 20))    # device memory is laid out once per layer
    return s


def _target(case):
    return int(math.floor(case["sparsity"] * case["rows"] * case["cols"] + 1e-9))


def _hessian(s):
    ctx, H = s["ctx"], s["H"]
    last = len(s["X"]) - 1
    for b, X in enumerate(s["X"]):
        ctx.obc_hessian(X, damp_rel=0.01 if b == last else -1.0, H=H, accumulate=b > 0)
    return H


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "calibrate":
        return {"Hinv": ctx.obc_invert(_hessian(s))}
    if kind == "refit":
        H = _hessian(s)
        ctx.obc_cross(s["X"][0], s["Y"], C=s["C"])
        W = ctx.obc_refit(H, s["C"], invert_in_place=True, W_out=s["Wfit"])
        return {"C": s["C"], "W": W, "Hinv": H}
    if kind == "layer":
        Hinv = ctx.obc_invert(_hessian(s))
        return dict(_prune(s, Hinv), Hinv=Hinv)
    if kind == "prune":
        return _prune(s, s["Hinv"])
    if kind == "blocks":
        W, Hinv = s["W"], s["Hinv"]
        r = ctx.obc_prune_blocks(W, Hinv, 4, want_trace=True)
        counts, mask = ctx.obc_global_select(r["loss"], r["order"], _target(case) // 4)
        What = ctx.obc_gather_trace(W, r["trace"], counts)
        return {"order": r["order"], "loss": r["loss"], "W": What, "counts": counts, "mask": mask}
    if kind == "quantize":
        W = s["W"]
        delta, offset, maxq = ctx.obc_minmax_grid(W, case["bits"], symmetric=case["symmetric"])
        r = ctx.obc_quant_rows(W, s["Hinv"], delta, offset, maxq, out=s["out"], outliers=case["outliers"])
        return {"order": r["order"], "loss": r["loss"], "codes": r["codes"], "W": r["W"], "delta": delta,
                "offset": offset}
    p = _prune(s, s["Hinv"])
    live = 1 - p["mask"]
    delta, offset, maxq = ctx.obc_minmax_grid(p["W"], case["bits"], live=live)
    q = ctx.obc_quant_rows(p["W"], s["Hinv"], delta, offset, maxq, live=live, out=s["quant"])
    return {"prune": p, "order": q["order"], "loss": q["loss"], "codes": q["codes"], "W": q["W"]}


def _prune(s, Hinv):
    case, ctx, W = s["case"], s["ctx"], s["W"]
    nm = (case["n"], case["m"]) if case.get("m") else (0, 0)
    r = ctx.obc_prune_rows(W, Hinv, k_steps=s["steps"], nm=nm, out=s["out"])
    if nm[1]:
        return {"order": r["order"], "loss": r["loss"], "W": r["W"]}
    counts, mask = ctx.obc_global_select(r["loss"], r["order"], _target(case))
    if r["trace"] is not None:
        What = ctx.obc_gather_trace(W, r["trace"], counts)
    else:
        What = ctx.obc_reconstruct_rows(W, Hinv, mask, max_pruned=int(counts.max()))
    return {"order": r["order"], "loss": r["loss"], "W": What, "counts": counts, "mask": mask}


# ------------------------------------------------------------------------------------------ account
def _eliminate(d, steps):
    """Operations of `steps` eliminations of one row from live size d: m^2 each (a multiply-add on one
    triangle of the symmetric matrix)."""
    cubes = lambda m: m * (m + 1) * (2 * m + 1) / 6.0  # noqa: E731
    return cubes(d) - cubes(d - steps)


def work(case):
    kind, d = case["kind"], case["cols"]
    R, N = case.get("rows", 0), case.get("samples", 0)
    if kind == "calibrate":
        return {"bytes": 4.0 * (d * N + d * d), "flops": float(d) * d * N + float(d) ** 3}
    if kind == "refit":
        return {"bytes": 4.0 * (d * N + R * N + d * d + 2 * R * d),
                "flops": float(d) * d * N + 2.0 * R * d * N + float(d) ** 3 + 2.0 * R * d * d}
    flops = 0.0
    nbytes = 4.0 * (R * d + d * d)
    if kind == "layer":
        flops += float(d) * d * N + float(d) ** 3
        nbytes += 4.0 * d * N
    if kind == "quantize":
        return {"bytes": nbytes + 16.0 * R * d, "flops": R * _eliminate(d, d)}
    steps = d // case["m"] * (case["m"] - case["n"]) if case.get("m") else d
    flops += R * _eliminate(d, steps)
    nbytes += R * (8.0 * steps + 4.0 * d)
    if kind == "blocks":
        nbytes = 4.0 * (R * d + d * d) + R * (8.0 * (d // 4) + 5.0 * d)
    elif not case.get("m"):
        nbytes += R * d
        if case.get("recover") == "closed" or kind == "compound":
            flops += R * (case["sparsity"] * d) ** 3 / 3.0
    if kind == "compound":
        left = int((1.0 - case["sparsity"]) * d)
        flops += R * (_eliminate(left, left) + float(left) ** 3)
        nbytes += 16.0 * R * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Four times what was measured.

    Front half, against torch in fp64: inverse and re-fitted weights 4e-6 .. 2.2e-5 (a Hessian rounded to
    fp32, condition number about 2e3), largest entry 1.4e-4 of the root mean square.

    Row solvers, the blocked against the rank-1 strategy (the same path with its sums in another order):
    weights agree to 2e-7 until two candidates are closer than the rounding of the matrix.  In pruning such a
    swap heals (1.7e-3 of the order entries, losses to 7e-3); in quantization the two weights may get other
    codes and everything after them in that row goes another way: about one row in 150 of 1500 .. 2300
    columns, of whose weights a tenth then sit on a neighbouring grid point (half a root mean square at 4 bit).
    """
    if case["kind"] in ("calibrate", "refit"):
        return {"rel": 1e-4, "max": 6e-4}
    if case["kind"] in ("quantize", "compound"):
        return {"rel": 0.03, "max": 0.99, "differ": 0.01}
    return {"rel": 0.028, "max": 0.99, "differ": 0.007}
