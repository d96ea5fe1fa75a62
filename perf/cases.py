"""Planner calls that are timed: what a user of the planner has it do, from a
290-candidate search to one over 3.9 million candidates.

A case names a model, a cluster, a search space and an objective; `prepare`
draws its synthetic inputs (layer profiles, compute tables, link bandwidths,
router counts) and keeps what a planning service keeps between calls: the
`Planner` with the problem image, the candidates and the result buffers in HBM.
One pass is `Planner.run`: cost tables, the stage DP of the objective and the
segmented arg-min with its plan.  All outputs are whole numbers (nanoseconds,
layer counts, masks) and have to be equal to the last bit.
"""
import math

import numpy as np
import torch

from paper_2609_39350_amd import binding

GB = 10**9
TP_VALUES = (1, 2, 4, 8)
CP_VALUES = (1, 2, 4, 8)

# Relative speed, memory (GB), compute efficiency of the device types, in the
# order in which a cluster of 2, 3 or 4 types takes them.
SPEED = {2: (1.0, 1.7), 3: (1.0, 1.4, 2.2), 4: (1.0, 1.3, 1.8, 2.5)}
MEMORY = {2: (16, 24), 3: (80, 64, 192), 4: (64, 96, 192, 288)}
EFF = {2: (1.0, 1.0), 3: (1.0, 0.9, 0.85), 4: (1.0, 0.95, 0.9, 0.85)}

# the three ways a pipeline's devices are laid out, besides block orderings (0)
SEQUENCES, DEVICE_COUNTS, WIDTHS = 1, 2, 3


def _case(name, **fields):
    case = {
        "name": name,
        "objective": "threshold",    # threshold | 1f1b | latency
        "stage_types": 0,            # 0 block orderings, 1 sequences, 2 device counts, 3 widths
        "once": False,               # a new problem on every pass: planner construction included
        "layers": 32, "dense_first": 0, "seq": 4096, "hidden": 4096, "experts": 64, "top_k": 8,
        "shared": 0, "ffn_dense": 14336, "ffn_expert": 2048, "zipf": 1.1,
        "counts": "32/16/16", "mem_scale": 1.0, "jitter": 0.05,
        "pp_max": 8, "ep_max": 64, "micro": "8/16/32", "mode": 0, "prune_window": 1,
        "recompute": True, "global_batch": 0,
    }
    case.update(fields)
    return case


_MOE61 = {"layers": 61, "dense_first": 3, "hidden": 7168, "experts": 256, "shared": 1, "ffn_dense": 18432,
          "counts": "64/64/64/64", "jitter": 0.15, "pp_max": 16, "micro": "16/32/64"}
_MOE96 = {"layers": 96, "seq": 8192, "hidden": 8192, "experts": 128, "top_k": 4, "ffn_dense": 28672,
          "ffn_expert": 4096, "counts": "256/256/256/256", "jitter": 0.15, "pp_max": 32, "ep_max": 128}


def listed():
    return [
        # the smallest search: 8 layers on 4 + 4 devices (latency and launches)
        _case("search_8l", layers=8, seq=2048, hidden=1024, experts=8, top_k=2, ffn_dense=4096, ffn_expert=3584,
              counts="4/4", pp_max=4, ep_max=8, micro="8"),
        # an ordinary search on a small cluster of three types
        _case("search_32l"),
        # a large model under tight memory, near-equal layers, strong router skew:
        # most candidates are infeasible or recompute
        _case("search_61l_tight", **dict(_MOE61, jitter=0.01, zipf=2.0, mem_scale=0.4)),
        # the largest search: every micro-batch count from 1 to 64
        _case("search_96l", **_MOE96, micro="1..64"),
        # odd sizes: 47 layers, groups that straddle device types, pipelines of 3, 6,
        # 12 and 24 stages, a fixed training batch
        _case("search_47l_odd", layers=47, experts=48, top_k=6, counts="40/24/32", pp_max=24, ep_max=48,
              micro="5/11/24/48", global_batch=48),
        # the 1F1B re-scoring of every candidate's (max, sum) frontier
        _case("frontier_61l", **_MOE61, objective="1f1b"),
        # the least 1F1B latency over every partition
        _case("latency_61l", **_MOE61, objective="latency"),
        _case("latency_96l", **_MOE96, micro="32/64", objective="latency"),
        # free device types per stage: every sequence as a candidate, and the DP over
        # device counts
        _case("sequences_32l", stage_types=SEQUENCES),
        _case("counts_61l", **_MOE61, stage_types=DEVICE_COUNTS),
        # data-parallel widths chosen per stage
        _case("widths_61l", **_MOE61, stage_types=WIDTHS),
        # a new problem planned once: from host tables to the plan, planner built anew
        _case("once_32l", once=True),
    ]


def draw(rng):
    """Another call of the same ranges: 6 to 96 layers, 2 to 4 device types in equal
    and unequal numbers, pipelines of up to 32 stages, any objective and layout."""
    largest = {}
    for case in listed():
        kind = _kind(case)
        largest[kind] = max(largest.get(kind, 0), work(case)["flops"])
    while True:
        kind = rng.choice(sorted(largest))
        types = rng.choice((2, 3, 4))
        unit = rng.choice((4, 8, 12, 16, 20, 24, 32, 40, 64, 128, 256))
        counts = [unit * rng.choice((1, 1, 2, 3)) // rng.choice((1, 1, 2)) for _ in range(types)]
        if sum(counts) > 1024:
            continue
        layers = round(6 * 16 ** rng.random())
        experts = rng.choice((8, 48, 64, 128, 256))
        top = rng.choice((1, 3, 8, 16, 64))
        micro = "1..%d" % top if rng.random() < 0.3 else "/".join(
            str(b) for b in sorted(rng.sample((2, 5, 8, 11, 16, 24, 32, 48, 64), rng.choice((1, 2, 3)))))
        case = _case(
            "", objective=kind if kind in ("1f1b", "latency") else "threshold",
            stage_types={"sequences": 1, "counts": 2, "widths": 3}.get(kind, 0), once=kind == "once",
            layers=layers, dense_first=rng.choice((0, 0, 1, 3)), seq=rng.choice((2048, 4096, 8192)),
            hidden=rng.choice((1024, 2048, 4096, 7168, 8192)), experts=experts, top_k=rng.choice((1, 2, 4, 8)),
            shared=rng.choice((0, 0, 1)), ffn_dense=rng.choice((4096, 14336, 18432)),
            ffn_expert=rng.choice((1024, 2048, 3584)), zipf=rng.choice((0.5, 1.1, 2.0)),
            counts="/".join(str(c) for c in counts), mem_scale=rng.choice((0.75, 1.0, 2.0)) * (4 if types == 2 else 1),
            jitter=rng.choice((0.01, 0.05, 0.15)), pp_max=rng.choice((3, 4, 8, 12, 16, 24, 32)),
            ep_max=rng.choice((8, 64, 128)), micro=micro, mode=1 if rng.random() < 0.1 else 0,
            # (windows off only where a sweep does not visit every stage cost)
            prune_window=rng.choice((1, 1, 1, 1, 2, 1 if kind == "latency" else 0)), recompute=rng.random() < 0.85)
        del case["name"]
        # weights, gradients and optimizer state leave room for activations in the cluster
        memory = sum(c * m for c, m in zip(counts, MEMORY[types])) * GB * case["mem_scale"]
        sizes = _problem(case, 0)["model"]
        if 18.0 * float(sizes["params_dense"].sum() + sizes["params_expert"].sum()) > 0.3 * memory:
            continue
        try:
            cost = work(case)["flops"]
        except binding.HapmoeError:   # a space the planner refuses (none, or too many sequences)
            continue
        if 0 < cost <= largest[kind]:
            return case


def _kind(case):
    if case["once"]:
        return "once"
    if case["stage_types"]:
        return ("", "sequences", "counts", "widths")[case["stage_types"]]
    return {"threshold": "search"}.get(case["objective"], case["objective"])


def _micro(case):
    text = case["micro"]
    if ".." in text:
        lo, hi = text.split("..")
        return list(range(int(lo), int(hi) + 1))
    return [int(b) for b in text.split("/")]


def _router_counts(rng, is_moe, experts, tokens, top_k, s):
    """Tokens per expert and layer: Zipf over shuffled experts, none above `tokens`."""
    n = len(is_moe)
    w = np.arange(1, experts + 1, dtype=np.float64)[None] ** -(s * rng.uniform(0.95, 1.05, size=(n, 1)))
    lo, hi = np.zeros((n, 1)), tokens * top_k / w[:, -1:] + 1.0
    for _ in range(60):   # the water level at which the layer routes tokens * top_k
        mid = 0.5 * (lo + hi)
        low = np.minimum(tokens, mid * w).sum(1, keepdims=True) < tokens * top_k
        lo, hi = np.where(low, mid, lo), np.where(low, hi, mid)
    counts = np.floor(np.minimum(tokens, hi * w)).astype(np.int64)
    return np.where(is_moe[:, None] != 0, rng.permuted(counts, axis=1), 0)


def _problem(case, seed):
    """The planner's host inputs: FLOP-derived compute tables with jitter, the usual
    Transformer parameter and activation sizes, random inter-type bandwidths."""
    rng = np.random.default_rng(seed)
    n, s, h, e, k = (case[f] for f in ("layers", "seq", "hidden", "experts", "top_k"))
    counts = [int(c) for c in case["counts"].split("/")]
    t = len(counts)
    is_moe = np.ones(n, dtype=np.uint8)
    is_moe[: min(case["dense_first"], n - 1)] = 0
    f_dense, f_exp = case["ffn_dense"], case["ffn_expert"]
    ffn = 6.0 * s * h * np.where(is_moe, f_exp, f_dense)
    total = 8.0 * s * h * h + 4.0 * s * s * h + ffn
    # forward and backward at 40 % of 1 PFLOP/s times the type's speed, split over
    # TP and CP with 5 % overhead a doubling: [type][tp][cp][layer]
    speed = np.array(SPEED[t])
    split = np.array([[(1.0 + 0.05 * math.log2(tp * cp)) / (tp * cp) for cp in CP_VALUES] for tp in TP_VALUES])
    scale = split[None, :, :, None] / speed[:, None, None, None] * (3.0 / 0.4e6)
    j = case["jitter"]
    dense = np.ceil(total * scale * rng.uniform(1 - j, 1 + j, size=(t, 4, 4, n))).astype(np.int64)
    expert = np.ceil(ffn * scale * rng.uniform(1 - j, 1 + j, size=(t, 4, 4, n))).astype(np.int64)
    bw = np.full((t, t), 400.0)
    for a in range(t):
        for b in range(a + 1, t):
            bw[a, b] = bw[b, a] = float(rng.integers(25, 51))
    alpha = np.full((t, t), 20000.0)
    np.fill_diagonal(alpha, 5000.0)
    return {
        "model": {
            "n_layers": n, "seq_len": s, "hidden": h, "n_experts": e, "top_k": k, "micro_batch_size": 1,
            "elem_bytes": 2, "moe_ffn_mult": float(k + case["shared"]), "is_moe": is_moe,
            "expert_tokens": _router_counts(rng, is_moe, e, s, k, case["zipf"]),
            "params_dense": np.where(is_moe, 4 * h * h + h * e + case["shared"] * 3 * h * f_exp,
                                     4 * h * h + 3 * h * f_dense).astype(np.int64),
            "params_expert": np.where(is_moe, e * 3 * h * f_exp, 0).astype(np.int64),
            "act_bytes": np.full(n, 34 * s * h, dtype=np.int64),
        },
        "cluster": {
            "n_types": t, "count": np.array(counts, dtype=np.int32),
            "speed": np.rint(100 * speed).astype(np.int32),
            "mem_bytes": np.array([int(m * GB * case["mem_scale"]) for m in MEMORY[t]], dtype=np.int64),
            "eff": np.array(EFF[t]), "route_coef": 6.0 * e / (0.4e6 * speed), "bw": bw, "alpha": alpha,
            "t_dense": dense, "t_ffn": np.minimum(expert, dense - 1),
        },
        "params": {"gamma": 0.5, "rc_time": 1.33, "rc_act": 0.4, "opt_coef": 0.01, "delta_num": 1, "delta_den": 5,
                   "eta_prune": 2, "prune_window": case["prune_window"], "prune_hetero": 1,
                   "allow_recompute": int(case["recompute"])},
        "space": {"pp_max": case["pp_max"], "tp_mask": 15, "cp_mask": 15, "ep_max": case["ep_max"], "tpe_mask": 15,
                  "mode": case["mode"], "micro": _micro(case), "stage_types": case["stage_types"],
                  "global_batch": case["global_batch"]},
    }


def prepare(case, seed):
    problem = _problem(case, seed)
    state = {"problem": problem, "objective": case["objective"], "planner": None}
    if not case["once"]:
        state["planner"] = binding.Planner(problem, "cuda:0")
    return state


def run(state):
    planner = state["planner"]
    if planner is None:
        planner = binding.Planner(state["problem"], "cuda:0")
    try:
        plan = planner.run(objective=state["objective"])
    except binding.HapmoeError as e:
        if e.code != -6:   # no candidate has a feasible partition: an answer too
            raise
        plan = {}
    out = {"results": planner.d_res, "config_best": planner.d_config_best,
           "plan": [plan.get(f, -1) for f in ("instance", "objective", "stage_sum", "t_max", "dp_const", "order",
                                              "n_micro")],
           "stages": np.array([plan.get(f, []) for f in ("layers", "stage_types", "recompute")], dtype=np.int64)}
    if planner.d_types is not None:
        out["types"] = planner.d_types
    if planner.d_widths is not None:
        out["all_widths"] = planner.d_widths
    return out


def _windows(case, pp):
    """Layers a stage may hold (how many values), as the case's window rule leaves them."""
    n = case["layers"]
    if case["prune_window"] == 0:
        return max(1, n - pp + 1)
    if case["prune_window"] == 2:
        return 2 if n % pp else 1
    return min(max(1, n - pp + 1), math.ceil(0.4 * n / pp) + 1)


def work(case):
    """Bytes: the problem in, the candidate list in, one result record a candidate out.
    Operations: one DP pass (at one threshold) of every pipeline the candidates name,
    six 32-bit operations a relaxation (cost against threshold, sum, minimum, in 64
    bits); sweeps over several thresholds are not counted."""
    problem = binding.HostProblem(_problem(case, 0))
    layout = binding.tables_layout(problem)
    n_cfg, n_ord, n_micro = layout["n_configs"], layout["n_orders"], len(_micro(case))
    n = n_cfg * n_ord * n_micro
    shapes = _problem(dict(case, micro="1", stage_types=case["stage_types"] if case["stage_types"] > 1 else 0), 0)
    cand = binding.enumerate_candidates(shapes)
    pps, configs = np.unique(cand["pp"], return_counts=True)
    configs = configs // max(1, len(cand) // max(1, n_cfg))
    counts = [int(c) for c in case["counts"].split("/")]
    relax = 0
    for pp, cfgs in zip((int(p) for p in pps), (int(c) for c in configs)):
        win = _windows(case, pp)
        nmax = case["layers"] - pp + 1   # end layers a stage can have
        band = [min(nmax, min(i, pp - i) * (win - 1) + 1) for i in range(1, pp + 1)]
        if case["stage_types"] == DEVICE_COUNTS:
            g = sum(counts) // pp
            k = [c // g for c in counts]
            level = [1]   # states (stages placed per type) of every level
            for m in k:
                level = np.convolve(level, np.ones(m + 1, dtype=np.int64))
            relax += cfgs * len(counts) * win * sum(int(level[i]) * band[i - 1] for i in range(1, pp + 1))
        elif case["stage_types"] == WIDTHS:
            units = [min(3 * i, 2 * pp - (pp - i)) - max(i, 2 * pp - 3 * (pp - i)) + 1 for i in range(1, pp + 1)]
            relax += cfgs * n_ord * 3 * win * sum(u * b for u, b in zip(units, band))
        else:
            orders = n_ord
            if case["stage_types"] == SEQUENCES:
                g = sum(counts) // pp
                orders = math.factorial(pp) // math.prod(math.factorial(c // g) for c in counts)
            relax += cfgs * orders * win * sum(band)
    nbytes = binding.image_bytes(problem) + n * (32 + 64) + 8 * n_cfg
    nbytes += 32 * n * {DEVICE_COUNTS: 1, WIDTHS: 2}.get(case["stage_types"], 0)
    return {"bytes": nbytes, "flops": 6 * relax * (n_micro if case["objective"] == "latency" else 1)}


def tolerance(case):
    """Whole nanoseconds, layers and masks: every bit of every record."""
    return "exact"


def exact(case, seed):
    """The outputs are whole numbers chosen by exact integer comparisons, compared bit
    for bit; a plain search over every partition in numpy takes minutes and more."""
    return None
