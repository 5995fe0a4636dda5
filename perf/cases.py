"""What is measured: the calls a scheduler makes of this library, over the range of cluster sizes.

A case is a dict of plain values.  Its "what" is the public call that one pass makes:

  round       Context.schedule_round          score every pair, match, prove (one scheduling interval)
  next round  Context.schedule_round_update   the following interval, a few workloads replaced
  typed round Context.schedule_round_typed    one predictor per GPU type
  scores      Context.score_pairs             every pair's score as float32 as well as the weights
  matching    Context.solve_assignment        a weight matrix the caller brings
  proof       Context.check_certificate, or check_certificate_noalloc with "graph" set

"law" names the feature law, predictor and scale of one of the synthetic configurations
(synth.CONFIGS); n and m are the numbers of online and offline workloads.
"""
import math

import numpy as np
import torch

import paper_2303_13803_amd as mm
import synth

CHURN = 0.02            # share of the workloads a following round has replaced (as in bench.py)
HIDDEN = (128, 64, 128)  # hidden widths of the per-GPU-type predictors
SLOW_LIMIT = 0.55       # slowdown of the online workload above which a pair is infeasible
SM = (2, 3)             # features the pair-dependent SM share is taken from


def listed():
    return [
        # one small cluster; what counts is launches, waits and host work
        {"name": "round 64x64", "what": "round", "law": "C1", "n": 64, "m": 64},
        # odd sizes: no dimension is a multiple of a tile, a wavefront or a vector
        {"name": "round 777x1501", "what": "round", "law": "C3", "n": 777, "m": 1501},
        # a thousand GPUs and as many jobs
        {"name": "round 1024x1024", "what": "round", "law": "C2", "n": 1024, "m": 1024},
        # more online than offline workloads: a short queue, solved on the transposed problem
        {"name": "round 3001x2003", "what": "round", "law": "C3", "n": 3001, "m": 2003},
        # a mid-sized cluster with a queue twice as long
        {"name": "round 4096x8192", "what": "round", "law": "C3", "n": 4096, "m": 8192},
        # the cluster of the paper's deployment: 20,000 GPUs (the benchmark's round)
        {"name": "round 20000x20000", "what": "round", "law": "C4", "n": 20000, "m": 20000},
        # the largest: a long queue, memory-hungry jobs (nine pairs in ten do not fit), 8-bit weights full of ties
        {"name": "round 20000x40000", "what": "round", "law": "C5", "n": 20000, "m": 40000},
        # the periodic invocation: two in a hundred workloads on each side replaced since the last round
        {"name": "next round 20000x20000", "what": "next round", "law": "C4", "n": 20000, "m": 20000},
        # three GPU generations, each with a predictor of its own
        {"name": "typed round 6001x9007", "what": "typed round", "law": "C4", "n": 6001, "m": 9007},
        # scores for inspection: every pair, unquantised, with the SM-share input and the slowdown limit
        {"name": "scores 4096x8192", "what": "scores", "law": "C3", "n": 4096, "m": 8192, "scale": 255.0, "options": True},
        # weights from elsewhere, one pair in ten feasible in no pattern
        {"name": "matching 20000x20000", "what": "matching", "n": 20000, "m": 20000, "high": 2 ** 24, "keep_one_in": 10},
        # re-verifying a plan and its duals, as an auditor of the scheduler does
        {"name": "proof 20000x40000", "what": "proof", "n": 20000, "m": 40000, "graph": False},
    ]


def _between(rng, low, high):
    """A whole number, its logarithm uniform."""
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    what = rng.choice(["round"] * 5 + ["next round", "typed round", "scores", "matching", "proof"])
    if what == "matching":
        n = _between(rng, 64, 20000)
        m = max(64, min(int(n * math.exp(rng.uniform(math.log(0.5), math.log(3.0)))), 400_000_000 // n))
        return {"what": what, "n": n, "m": m, "high": rng.choice([2 ** 20, 2 ** 24]), "keep_one_in": rng.choice([2, 4, 10])}
    if what == "proof":
        n = _between(rng, 64, 20000)
        return {"what": what, "n": n, "m": min(40000, int(n * rng.uniform(1.0, 3.0))), "graph": rng.random() < 0.5}
    if what == "typed round":
        law = rng.choice(["C3", "C4"])
    else:
        law = rng.choice(["C2", "C3", "C4", "C5"])
    n = _between(rng, 64, 20000)
    # the queue is about as long as the cluster is large; memory-hungry jobs (C5) wait in longer ones
    wide = rng.uniform(1.5, 3.0) if law == "C5" else math.exp(rng.uniform(math.log(0.5), math.log(3.0)))
    m = max(64, min(int(n * wide), (800_000_000 if law == "C5" else 400_000_000) // n))
    c = {"what": what, "law": law, "n": n, "m": m}
    if what == "scores":                # every pair goes through the predictor: a sixth of the largest matrix at most
        c["n"], c["m"] = min(n, 8000), min(m, 8000)
        c["scale"] = 255.0
        c["options"] = rng.random() < 0.5
    return c


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _weights(n, m):
    """The caller's weight matrix: rows padded to whole 16-byte groups."""
    return torch.zeros((n, (m + 3) // 4 * 4), dtype=torch.int32, device="cuda")


def _plan(s, n, m):
    s["row2col"] = torch.empty(n, dtype=torch.int32, device="cuda")
    s["u"] = torch.empty(n, dtype=torch.int64, device="cuda")
    s["v"] = torch.empty(m, dtype=torch.int64, device="cuda")


def _planted_proof(s, n, m, seed):
    """A matrix with a known optimal matching and duals: W = a_i + b_j - slack, slack 0 on the planted
    pairs and at least 0 elsewhere, one pair in five infeasible; u = K a, v = K b, b = 0 where unmatched."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    ints = lambda high, shape: torch.randint(0, high, shape, generator=gen, device="cuda", dtype=torch.int32)
    cols = torch.randperm(m, generator=gen, device="cuda")[:n]
    a, b = ints(1 << 22, (n,)) + (1 << 23), torch.zeros(m, dtype=torch.int32, device="cuda")
    b[cols] = ints(1 << 22, (n,))
    W = _weights(n, m)
    for i0 in range(0, n, 2048):
        i1 = min(n, i0 + 2048)
        w = a[i0:i1, None] + b[None, :] - ints(1 << 23, (i1 - i0, m))
        w[ints(5, (i1 - i0, m)) == 0] = mm.INFEASIBLE
        W[i0:i1, :m] = w
    W[torch.arange(n, device="cuda"), cols] = a + b[cols]
    s["W"], s["row2col"], s["K"] = W, cols.to(torch.int32), min(n, m) + 1
    s["u"], s["v"] = a.to(torch.int64) * s["K"], b.to(torch.int64) * s["K"]


def prepare(case, seed):
    what, n, m = case["what"], case["n"], case["m"]
    s = {"what": what, "n": n, "m": m}
    if what == "proof":
        _planted_proof(s, n, m, seed)
        if case["graph"]:               # no context is needed: the result goes to a buffer on the device
            s["out"] = torch.zeros(64, dtype=torch.uint8, device="cuda")
        else:
            s["ctx"] = mm.Context(n, m)
        return s
    s["ctx"] = ctx = mm.Context(n, m)
    _plan(s, n, m)
    if what == "matching":
        s["W"] = synth.device_masked_matrix(seed, n, m, case["high"], case["keep_one_in"])
        return s
    r = synth.scheduling_round(case["law"], seed, n, m)
    F, H, scale = r["cfg"].F, r["cfg"].H, case.get("scale", r["cfg"].scale)
    s["W"] = _weights(n, m)
    if what == "typed round":
        s["params"] = [{k: _dev(v) for k, v in p.items()} for p in synth.typed_predictors(seed, F, HIDDEN)]
        s["preds"] = [ctx.predictor(p, scale) for p in s["params"]]
        s["types"] = _dev(synth.gpu_types(seed, n, len(HIDDEN)))
    elif what == "scores" and case["options"]:
        params = {k: _dev(v) for k, v in synth.with_slowdown_unit(r["params"], seed).items()}
        params["W1sm"] = _dev(synth.with_sm_input(r["params"], seed)["W1"][:, -1])
        s["pred"] = ctx.predictor(params, scale, sm=SM, slow_limit=SLOW_LIMIT)
    else:
        s["pred"] = ctx.predictor({k: _dev(v) for k, v in r["params"].items()}, scale)
    if what == "scores":
        s["sigma"] = torch.zeros((n, m), dtype=torch.float32, device="cuda")
    if what == "next round":
        # the matrix of the previous interval is in hand; then some workloads end and others take their place
        ctx.score_pairs(s["pred"], _dev(r["x_on"]), _dev(r["x_off"]), s["W"])
        fresh = synth.scheduling_round(case["law"], seed + 500_000_000, n, m)
        rows = np.sort(synth.permutation(seed, n, 3)[:max(1, int(CHURN * n))]).astype(np.int32)
        cols = np.sort(synth.permutation(seed, m, 4)[:max(1, int(CHURN * m))]).astype(np.int32)
        r["x_on"][rows], r["x_off"][cols] = fresh["x_on"][rows], fresh["x_off"][cols]
        s["rows"], s["cols"] = _dev(rows), _dev(cols)
    s["x_on"], s["x_off"] = _dev(r["x_on"]), _dev(r["x_off"])
    return s


# Which of the optimal matchings a solve returns, and which optimal duals, is not determined (and differs
# from pass to pass): what is compared of it is the optimum and that its proof verified on the device.
def run(s):
    what, n, m = s["what"], s["n"], s["m"]
    if what == "proof":
        if "out" in s:
            rc = mm.binding.check_certificate_noalloc(s["W"], n, m, s["row2col"], s["u"], s["v"], s["K"], s["out"])
            return {"certificate": s["out"], "rc": rc}
        c = s["ctx"].check_certificate(s["W"], n, m, s["row2col"], s["u"], s["v"], s["K"])
        return {"primal": c.primal, "dual": c.dual, "least": c.min_reduced_cost, "matched": c.matched, "proved": c.cert_ok}
    plan = (s["row2col"], s["u"], s["v"])
    if what == "scores":
        s["ctx"].score_pairs(s["pred"], s["x_on"], s["x_off"], s["W"], s["sigma"])
        return {"weights": s["W"], "sigma": s["sigma"]}
    if what == "matching":
        res = s["ctx"].solve_assignment(s["W"], n, m, *plan)
        return {"total": res.primal, "proved": res.cert_ok}
    if what == "round":
        res = s["ctx"].schedule_round(s["pred"], s["x_on"], s["x_off"], s["W"], *plan)
    elif what == "next round":
        res = s["ctx"].schedule_round_update(s["pred"], s["x_on"], s["x_off"], s["rows"], s["cols"], s["W"], *plan)
    else:
        res = s["ctx"].schedule_round_typed(s["preds"], s["types"], s["x_on"], s["x_off"], s["W"], *plan)
    return {"weights": s["W"], "total": res.primal, "proved": res.cert_ok}


def work(case):
    what, n, m = case["what"], case["n"], case["m"]
    pairs = n * m
    duals = 12 * n + 8 * m                              # row2col, u, v
    if what in ("proof", "matching"):
        return {"bytes": 4 * pairs + duals, "flops": 0}
    cfg = synth.CONFIGS[case["law"]]
    features = 4 * cfg.F * (n + m)
    masked = 0.5 if cfg.masked is None else cfg.masked  # (uniform memory fractions left as drawn: every second pair fits)
    if what == "scores":
        return {"bytes": 8 * pairs + features, "flops": 2 * cfg.H * cfg.H * pairs}
    if what == "next round":                            # the changed lines, and the matrix read once to match
        scored = (1 - (1 - CHURN) ** 2) * pairs
        return {"bytes": 4 * pairs + 4 * scored + features + duals, "flops": 2 * cfg.H * cfg.H * (1 - masked) * scored}
    hidden = cfg.H * cfg.H
    if what == "typed round":                           # types in shares 1, 1/2, 1/3
        share = [1 / (t + 1) for t in range(len(HIDDEN))]
        hidden = sum(s * h * h for s, h in zip(share, HIDDEN)) / sum(share)
    return {"bytes": 4 * pairs + features + duals, "flops": 2 * hidden * (1 - masked) * pairs}


def tolerance(case):
    if case["what"] == "scores":
        # float32 sums through two layers and a logistic; a weight may round to the next of its 256 levels
        return {"rel": 1e-5, "max": 1e-4, "differ": 1e-3}
    return "exact"                                      # whole numbers throughout
