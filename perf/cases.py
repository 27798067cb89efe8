"""The work that is timed for this framework: what a user has one BrownoutMoE layer do, through the public calls of
`paper_2507_17133_amd.binding`.

A case names a layer shape of `workloads.CONFIGS` (Mixtral-8x7B-, Qwen3-30B-A3B-, DeepSeek-V3-, Qwen1.5-MoE-shaped, or
the tiny one) and a task:

  forward  one `moe_forward` over T tokens: prefill with thousands of tokens, a chunk of a prefill, a decode batch with
           one token per request, a single request; `fraction` is the brownout fraction f (threshold 1 - f) that the
           latency controller has chosen, `full` drops the delegated tokens instead of serving them by united experts,
           `packed` says whether the program repacked its gate once (a serving program) or passes the fp32 matrix,
           `own_route` that it calls `moe_route` first and hands the row lists to `moe_forward` (a program that looks
           at the expert counts or keeps the routing for its statistics)
  route    `moe_route` alone, all routing artefacts wanted
  build    `moe_build_united` with the distillation loss evaluated on T calibration tokens
  distill  `moe_build_united`, then `moe_distill_united` with `steps` Adam steps on T calibration tokens (forward and
           backward pass), the way united experts are made for a model; `experts` of the layer, `way` of them per group
"""
import math

import numpy as np
import torch

from paper_2507_17133_amd import binding as B
from paper_2507_17133_amd.workloads import CONFIGS, make_gate

#: Most tokens of a drawn batch and of a drawn calibration set, per layer shape: what the repository's benchmark
#: configurations run, and for the DeepSeek-V3 shape a size whose zero-brownout pass costs less than the listed one.
MOST_TOKENS = {"tiny": 1024, "mixtral_prefill": 4096, "qwen3_30b_a3b": 8192, "deepseek_v3": 9000, "qwen15_moe_a27b": 8192}
MOST_CALIB = 2048


def _forward(name, layer, T, fraction, full=False, packed=True, own_route=False, residual=False, way=8):
    return {"name": name, "task": "forward", "layer": layer, "T": T, "fraction": fraction, "full": full,
            "packed": packed, "own_route": own_route, "residual": residual, "way": way}


def listed():
    return [
        # the smallest call: a layer of toy size, fp32 gate; five launches and the host call are all there is
        _forward("tiny_64", "tiny", 64, 0.25, packed=False),
        # one request decoding alone: top-8 of 128 small experts, the launches' latency against 75 MB of weights
        _forward("qwen3_decode_1", "qwen3_30b_a3b", 1, 0.0),
        # a small decode batch of the paper's 60-expert model at its setting (8, 0.4); a shared expert of its own width
        _forward("qwen15_decode_37", "qwen15_moe_a27b", 37, 0.6),
        # the benchmark's decode batch: every expert's weights streamed once, 64 rows each
        _forward("mixtral_decode_256", "mixtral_prefill", 256, 0.0),
        # the same batch when the controller has browned out everything: one dense united expert
        _forward("mixtral_decode_256_united", "mixtral_prefill", 256, 1.0),
        # a chunk of a prefill, an odd number of tokens: 257 units, most of them with few rows
        _forward("deepseek_chunk_1021", "deepseek_v3", 1021, 0.4),
        # routing by itself, as a program calls it that plans batches on the expert counts
        {"name": "qwen3_route_3001", "task": "route", "layer": "qwen3_30b_a3b", "T": 3001, "fraction": 0.5, "full": False,
         "packed": True, "way": 8},
        # prefill of the 60-expert model with the caller's own routing, full brownout and the residual added
        _forward("qwen15_prefill_5003_full", "qwen15_moe_a27b", 5003, 0.8, full=True, own_route=True, residual=True, way=4),
        # the three prefill batches of the benchmark
        _forward("mixtral_prefill_4096", "mixtral_prefill", 4096, 0.3),
        _forward("qwen3_prefill_8192", "qwen3_30b_a3b", 8192, 0.5),
        _forward("deepseek_prefill_16384", "deepseek_v3", 16384, 0.4),
        # making united experts for the 60-expert model's shape: a full group and a ragged one, some steps of training
        {"name": "qwen15_distill_2048", "task": "distill", "layer": "qwen15_moe_a27b", "T": 2048, "experts": 12, "way": 8,
         "steps": 8},
    ]


def _log_uniform(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    task = rng.choice(["forward"] * 5 + ["route", "build", "distill"])
    layer = rng.choice(["tiny", "mixtral_prefill", "qwen3_30b_a3b", "deepseek_v3", "qwen15_moe_a27b"])
    if task in ("forward", "route"):
        T = _log_uniform(rng, 1, MOST_TOKENS[layer])
        case = _forward("", layer, T, rng.choice([0.0, 0.0, 0.25, 0.3, 0.4, 0.5, 0.6, 0.75, 0.8, 1.0]), full=rng.random() < 0.15,
                        packed=rng.random() < 0.75, own_route=rng.random() < 0.2, residual=rng.random() < 0.3,
                        way=rng.choice([2, 4, 8, 8]))
        if task == "route":
            case = {k: v for k, v in case.items() if k not in ("own_route", "residual")}
            case["task"] = "route"
        del case["name"]
        return case
    # offline work: shapes whose experts a calibration batch is run through one by one
    layer = rng.choice(["tiny", "qwen3_30b_a3b", "qwen15_moe_a27b"])
    if task == "build":
        return {"task": "build", "layer": layer, "T": _log_uniform(rng, 64, MOST_CALIB), "way": rng.choice([2, 4, 8])}
    return {"task": "distill", "layer": layer, "T": 64 * _log_uniform(rng, 2, MOST_CALIB // 64), "experts": rng.randint(4, 16),
            "way": rng.choice([2, 4, 8]), "steps": rng.randint(2, 10)}


def _layer(case):
    c = CONFIGS[case["layer"]]
    more = {"T": case["T"], "way": case["way"], "zipf_s": c.zipf_s}
    if case["task"] in ("build", "distill"):
        more.update(n_shared=0, F_s=0, m=case.get("experts", c.m))
        more["K"] = min(c.K, more["m"])
    elif case["layer"] == "mixtral_prefill" and case["T"] <= 256:
        more["zipf_s"] = None            # the decode configuration: uniform gate
    return c.with_(**more)


def _weights(n, d, F, gen):
    """n SwiGLU experts, N(0, 1/d) in bf16 (the distribution of `workloads.make_ffn_weights`, drawn in place)."""
    std = 1.0 / math.sqrt(d)
    return tuple(torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)
                 for s in ((n, F, d), (n, F, d), (n, d, F)))


def prepare(case, seed):
    L = _layer(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 1000 + 17)
    s = {"case": case, "threshold": 1.0 - case.get("fraction", 0.0)}
    x = torch.empty((L.T, L.d), dtype=torch.bfloat16, device="cuda").normal_(0.0, 1.0, generator=gen)
    s["x"] = x
    cfg = B.config_of(L)
    cfg.add_residual = 1 if case.get("residual") else 0
    if case["task"] == "route" or case["task"] == "forward":
        gate_w, s["gate_b"], _ = make_gate(L, seed, "cuda")
        if case["packed"]:
            s["gate"] = B.pack_gate(cfg, gate_w)
            cfg = B.with_packed_gate(cfg)
        else:
            s["gate"] = gate_w
        s["workspace"] = B.alloc_workspace(cfg, L.T)
    if case["task"] == "route" or case.get("own_route"):
        s["route"] = B.alloc_route_out(cfg, L.T)
        s["route"].row_token.zero_()      # entries past n_rows are not written
        s["route"].row_weight.zero_()
    if case["task"] != "route":
        s["experts"] = _weights(L.m, L.d, L.F, gen)
    if case["task"] == "forward":
        s["united"] = _weights(L.G, L.d, L.F, gen) if s["threshold"] < 1.0 and not case["full"] else None
        s["shared"] = _weights(L.n_shared, L.d, L.F_s, gen) if L.n_shared else None
        s["out"] = torch.empty_like(x)
    elif case["task"] == "build":
        s["workspace"] = B.alloc_workspace(cfg, L.T)
    s["cfg"] = cfg
    return s


def run(s):
    case, cfg = s["case"], s["cfg"]
    if case["task"] == "forward":
        route = None
        if case["own_route"]:
            route = B.moe_route(cfg, s["x"], s["gate"], s["gate_b"], s["threshold"], case["full"], out=s["route"],
                                workspace=s["workspace"])
        return B.moe_forward(cfg, s["x"], s["gate"], s["gate_b"], s["experts"], s["united"], s["shared"], s["threshold"],
                             case["full"], route=route, out=s["out"], workspace=s["workspace"])
    if case["task"] == "route":
        r = B.moe_route(cfg, s["x"], s["gate"], s["gate_b"], s["threshold"], case["full"], out=s["route"],
                        workspace=s["workspace"])
        return vars(r)
    if case["task"] == "build":
        united, loss = B.moe_build_united(cfg, s["experts"], s["x"], workspace=s["workspace"])
        return {"united": united, "loss": loss}
    united, _ = B.moe_build_united(cfg, s["experts"])
    history = B.moe_distill_united(cfg, s["experts"], united, s["x"], case["steps"], 1e-4)
    return {"united": united, "history": history}


def _rows_and_units(L, case):
    """Rows of the FFN GEMMs and units that hold rows, for a typical draw: the gate's logits are close to
    ln p_i + Gumbel noise, so top-K of such a draw gives the counts, and the decision is taken on them."""
    T = min(L.T, 4096)
    rng = np.random.default_rng(1)
    logp = np.zeros(L.m) if L.zipf_s is None else -L.zipf_s * np.log(rng.permutation(L.m) + 1.0)
    top = np.argpartition(-(logp + rng.gumbel(size=(T, L.m))), L.K - 1, axis=1)[:, :L.K]
    cnt = np.bincount(top.ravel(), minlength=L.m)
    order = np.argsort(-cnt, kind="stable")
    before = np.cumsum(cnt[order]) - cnt[order]
    s2 = np.zeros(L.m, bool)
    s2[order] = before >= T * L.K * (1.0 - case["fraction"])
    unit = np.arange(L.m)
    for g in range(L.G):
        held = [i for i in range(g * L.way, min(L.m, (g + 1) * L.way)) if s2[i] and cnt[i] > 0]
        if case["full"]:
            unit[held] = -1
        elif len(held) >= 2:
            unit[held] = L.m + g
    of = unit[top]
    pairs = np.unique((np.arange(T)[:, None] * (2 * L.m + 1) + of)[of >= 0])
    return len(pairs) * L.T // T, len(set(pairs % (2 * L.m + 1)))


def work(case):
    L = _layer(case)
    expert = 3 * L.d * L.F * 2                               # bytes of one expert's weights
    if case["task"] == "build":
        # every expert and every united expert on the calibration tokens; the weights read once, the means written
        n = L.m + L.G
        return {"bytes": n * expert + L.T * L.d * 2, "flops": 6 * n * L.T * L.d * L.F}
    if case["task"] == "distill":
        trained = sum(1 for g in range(L.G) if min(L.m, (g + 1) * L.way) - g * L.way > 1)
        # teachers once; a step is three products forward and four backward, the last evaluation is forward only
        flops = 6 * L.m * L.T * L.d * L.F + trained * (14 * case["steps"] + 6) * L.T * L.d * L.F
        # the optimiser's state (fp32 master weights and two moments) is read and written in every step
        return {"bytes": L.m * expert + trained * case["steps"] * 3 * L.d * L.F * 24, "flops": flops}
    gate = {"bytes": L.T * L.d * 2 + L.m * L.d * 4, "flops": 2 * L.T * L.d * L.m}
    if case["task"] == "route":
        return {"bytes": gate["bytes"] + L.T * L.K * 20, "flops": gate["flops"]}
    rows, units = _rows_and_units(L, case)
    shared = L.n_shared * 3 * L.d * L.F_s
    return {"bytes": gate["bytes"] + units * expert + 2 * shared + L.T * L.d * 2,
            "flops": gate["flops"] + 6 * rows * L.d * L.F + 2 * L.T * shared}


def tolerance(case):
    if case["task"] == "route":
        # fp32 weights of the winners: 8e-8 (largest 4e-7) from 64-bit arithmetic; whole numbers stay the same
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
    if case["task"] == "forward":
        # bf16 H and out, half-precision Y: 2.4e-3 (largest 0.011 to 0.017) from the layer equation in 64 bits
        return {"rel": 1e-2, "max": 0.06}
    if case["task"] == "build":
        # the loss is 7e-4 from its 64-bit value (half-precision rows rounded toward zero); the means are exact
        return {"rel": 3e-3, "max": 1e-2}
    # trained weights in bf16 and the loss before every step: 2.2e-3 (largest 0.11: an Adam step is a step of full
    # size whichever sign a gradient near zero has) and 1e-3 from the same training in 64 bits
    return {"rel": 8e-3, "max": 0.4}
