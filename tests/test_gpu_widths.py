"""Per-stage data-parallel widths on the GPU (hapmoe_stage_dp_widths) against
the oracle, through the C ABI: status, objective, stage sum, largest stage,
recomputation mask, stage lengths, stage type sets and widths bit-exact."""
import copy

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2609_39350_amd import binding, workloads
from tests import parity_digest
from tests.problems import worked_problem_w2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


def widths(p, **kw):
    q = copy.deepcopy(p)
    q["space"]["stage_types"] = 3
    for k, v in kw.items():
        q["params"][k] = v
    return q


def compare(problem, pl, idx, ref=None):
    res, types, wd = pl.results(), pl.stage_types(), pl.widths()
    if ref is None:
        o = orc.Oracle(problem)
        ref = [o.solve(int(i)) for i in idx]
    bad, feasible = [], 0
    for i, r in zip(idx, ref):
        g = res[i]
        if int(g["status"]) != r["status"]:
            bad.append((int(i), "status", int(g["status"]), r["status"]))
            continue
        if r["status"]:
            assert not types[i].any() and not wd[i].any()
            continue
        feasible += 1
        pp = r["pp"]
        got = (int(g["objective"]), int(g["stage_sum"]), int(g["t_max"]), list(g["layers"][:pp]),
               [(int(g["recompute_mask"]) >> s) & 1 for s in range(pp)], [int(x) for x in types[i][:pp]],
               [int(x) for x in wd[i][:pp]])
        exp = (r["opt"], r["sum"], r["tmax"], r["layers"], r["recompute"], r["stage_mask"], r["width"])
        if got != exp:
            bad.append((int(i), got, exp))
    assert not bad, f"{len(bad)} mismatches, first: {bad[:3]}"
    return feasible


def _run(p):
    pl = binding.Planner(p, "cuda:0")
    plan = pl.run()
    return pl, plan


def test_worked_problem_and_config1_every_candidate(torch):
    for p in (widths(worked_problem_w2()), widths(workloads.config(1))):
        print(f"widths: {p['name']}", flush=True)
        pl, plan = _run(p)
        assert compare(p, pl, range(pl.n)) > 0
        res = pl.results()
        obj = np.where(res["status"] == 0, res["objective"], np.iinfo(np.int64).max)
        assert plan["instance"] == int(np.argmin(obj)) and plan["objective"] == int(obj.min())
        assert sum(plan["widths"]) == 2 * plan["config"][0]


def test_random_tiny_every_candidate(torch):
    total = 0
    for s in range(16):
        p = widths(workloads.random_tiny(700 + s, n_layers=int(4 + s % 6), max_pp=4))
        try:
            orc.Oracle(p)
        except ValueError:
            continue
        print(f"widths: {p['name']}", flush=True)
        pl = binding.Planner(p, "cuda:0")
        pl.eval_cost_tables()
        pl.stage_dp()
        total += compare(p, pl, range(pl.n))
    assert total > 30


@pytest.mark.parametrize("window", [1, 0])
def test_config2_sampled(torch, window):
    p = widths(workloads.config(2), prune_window=window)
    print(f"widths: config 2, windows {window}", flush=True)
    pl, plan = _run(p)
    idx = sorted(set(list(range(3, pl.n, max(1, pl.n // 160))) + [plan["instance"]]))
    from tests.test_gpu_parity import oracle_many
    assert compare(p, pl, idx, ref=oracle_many(p, idx, pool=True)) > 0


def test_config2_every_candidate(torch):
    """Every candidate of configuration 2 (10,584, one launch) against stored
    oracle digests of status, objective, stage sum, largest stage,
    recomputation mask, stage lengths, stage type sets and widths
    (tests/golden/parity_refs.npz, written from oracle/ alone)."""
    import os
    refs_path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "parity_refs.npz")
    with np.load(refs_path) as f:
        if "cfg2_widths" not in f.files:
            pytest.skip("no per-stage widths references in parity_refs.npz")
        idx, ref = f["cfg2_widths_idx"], f["cfg2_widths"]
    p = widths(workloads.config(2))
    print("widths: config 2, every candidate against stored oracle digests", flush=True)
    pl, plan = _run(p)
    assert len(idx) == pl.n
    got = parity_digest.of_gpu(pl.results(), idx, pl.stage_types(), pl.widths())
    bad = np.nonzero(got != ref)[0]
    assert len(bad) == 0, f"{len(bad)} of {len(idx)} differ, first: {idx[bad][:5]}"
    assert (pl.results()["status"] == 0).sum() > 1000


def test_config2_sub_ranges_equal_one_launch(torch):
    p = widths(workloads.config(2))
    pl, _ = _run(p)
    whole = (pl.results().copy(), pl.stage_types().copy(), pl.widths().copy())
    pl.d_res.zero_()
    pl.d_types.zero_()
    pl.d_widths.zero_()
    cuts = [0, 1, 2500, 2500, 7001, pl.n]
    for a, b in zip(cuts[:-1], cuts[1:]):
        pl.stage_dp(first=a, count=b - a)
    assert np.array_equal(pl.results(), whole[0])
    assert np.array_equal(pl.stage_types(), whole[1]) and np.array_equal(pl.widths(), whole[2])


def test_config3_launch_and_shallow_sample(torch):
    """The 61-layer workload in width mode (93,888 candidates, one launch); the
    oracle on a sample of the pipelines of up to 4 stages, and the properties of
    every result."""
    p = widths(workloads.config(3))
    print("widths: config 3", flush=True)
    pl, plan = _run(p)
    res, wd = pl.results(), pl.widths()
    ok = res["status"] == 0
    pp = pl.cand_host["pp"]
    assert (wd[ok].astype(int).sum(axis=1) == 2 * pp[ok]).all()
    assert (res["layers"][ok].astype(int).sum(axis=1) == p["model"]["n_layers"]).all()
    shallow = np.nonzero(pp <= 4)[0]
    idx = sorted(set(shallow[:: max(1, len(shallow) // 120)].tolist()))
    from tests.test_gpu_parity import oracle_many
    assert compare(p, pl, idx, ref=oracle_many(p, idx, pool=True)) > 0


def _numpy_sweep(cost, micro):
    """Least sum + (B-1) max over the width sequences and partitions on an explicit cost
    tensor [pp][2pp+1][3][n+1][n+1]: (objective, sum, largest stage), the least largest
    stage on ties, by passes at descending thresholds from infinity.  A pass keeps the
    least (sum, largest stage) of every state, which a longer path keeps in order."""
    big = np.int64(1) << 60
    pp, units, _, w1, _ = cost.shape
    cost = np.minimum(cost, big)

    def least_sum(t):
        f, m = np.full((units, w1), big), np.full((units, w1), big)
        f[0, 0] = m[0, 0] = 0
        for s in range(pp):
            g, h = np.full((units, w1), big), np.full((units, w1), big)
            for w in (1, 2, 3):
                for u in range(units - w):
                    if f[u].min() == big:
                        continue
                    c = cost[s, u, w - 1]
                    v = np.where(c <= t, np.minimum(f[u][:, None] + c, big), big)
                    least = v.min(axis=0)
                    mx = np.where(v == least, np.maximum(m[u][:, None], c), big).min(axis=0)
                    better = (least < g[u + w]) | ((least == g[u + w]) & (mx < h[u + w]))
                    g[u + w], h[u + w] = np.where(better, least, g[u + w]), np.where(better, mx, h[u + w])
            f, m = g, h
        return int(f[units - 1, w1 - 1]), int(m[units - 1, w1 - 1])

    best, t = None, int(big) - 1
    while t >= 0:
        f, mx = least_sum(t)
        if f >= big:
            break
        obj = f + (micro - 1) * mx
        if best is None or obj <= best[0]:
            best = (obj, f, mx)
        # a lower threshold has a sum >= f
        t = min(mx - 1, (best[0] - f) // (micro - 1)) if micro > 1 else (mx - 1 if f == best[0] else -1)
    return best


@pytest.mark.parametrize("layers,pp", [(100, 16), (33, 8)])
def test_no_windows_against_dense_sweep(torch, layers, pp):
    """No pruning-1 windows, so that every (level, half-groups) row has the widest band:
    at 100 layers and 16 stages the state lists and intervals exceed a workgroup's LDS
    and lie in the workspace (the second work list is not empty), at 33 and 8 they do
    not.  Whole numbers: every value equal."""
    p = widths(workloads.random_tiny(61, n_layers=layers, n_types=2, max_pp=pp, micro=[2 * pp]), prune_window=0)
    p["cluster"]["count"] = np.array([2 * pp, 2 * pp], dtype=np.int32)
    p["cluster"]["mem_bytes"] = np.array([60, 90], dtype=np.int64) * 10**9
    p["space"].update(pp_max=pp, tp_mask=1, cp_mask=1, tpe_mask=1, ep_max=1)
    print(f"widths: {layers} layers, {pp} stages, no windows", flush=True)
    pl, _ = _run(p)
    o, res = orc.Oracle(p), pl.results()
    idx = [int(i) for i in np.nonzero((pl.cand_host["pp"] == pp) & (res["status"] == 0))[0]][:1]
    assert idx
    in_ws = int(pl.d_dp_ws[4:8].cpu().numpy().view(np.uint32)[0])
    assert (in_ws > 0) == (layers == 100)
    for i in idx:
        got = tuple(int(res[i][f]) for f in ("objective", "stage_sum", "t_max"))
        cost, _ = o.width_costs(i)
        ref = _numpy_sweep(cost, int(pl.cand_host["n_micro"][i]))
        const = got[0] - got[1] - (int(pl.cand_host["n_micro"][i]) - 1) * got[2]
        assert got == (ref[0] + const, ref[1], ref[2])
        cfg, order = i // (o.n_orders() * 1), i % o.n_orders()
        assert const == o.dp_const(o.configs()[cfg], order)


def _overflows(o, n_layers, n_types, cfg, masks):
    """A term of some width on one of the device-type sets reaches the 2^44 limit."""
    big = 2.0 ** 44
    for w in (1, 2, 3):
        for m in masks:
            for layer in range(n_layers):
                t = o.width_terms(cfg, layer, m, w)
                x = [t["mask"][f] for f in ("a2a", "tp", "cp", "t_r1")] + [t["mem"][f] for f in ("w", "a0")]
                x += [t["type"][h][f] for h in range(n_types) for f in ("comp", "expert")]
                if max(x) >= big:
                    return True
    return False


def test_overflow_of_any_type_set(torch):
    """A configuration is refused (OVERFLOW) if a term of any device-type set leaves the
    range, also of a set that no stage can hold: the all-to-all of the three types
    takes the latency of one link and the bandwidth of another, and only with both does
    it pass 2^44.  Six stages of four devices hold at most two of the types of eight."""
    p = widths(workloads.random_tiny(5, n_layers=8, n_types=3, max_pp=6, micro=[4, 9]))
    m, c = p["model"], p["cluster"]
    m.update(seq_len=512, hidden=256, n_experts=4, top_k=2, micro_batch_size=1, elem_bytes=2)
    m["is_moe"][:] = 1
    m["expert_tokens"] = np.full((8, 4), 256, dtype=np.int64)
    m["params_expert"] = np.full(8, 10**6, dtype=np.int64)
    c["count"] = np.array([8, 8, 8], dtype=np.int32)
    c["mem_bytes"] = np.full(3, 10**14, dtype=np.int64)
    c["alpha"], c["bw"] = np.full((3, 3), 1000.0), np.full((3, 3), 100.0)
    part = 0.15 * 2.0 ** 44   # four exchanges of either part alone stay below, of both together do not
    c["alpha"][0, 1] = c["alpha"][1, 0] = part
    c["bw"][1, 2] = c["bw"][2, 1] = 512 * 2 * 256 * 2 / part
    p["params"].update(gamma=0.0, prune_window=0, prune_hetero=0, allow_recompute=1, rc_time=1.33)
    p["space"].update(pp_max=6, tp_mask=1, cp_mask=1, tpe_mask=1, ep_max=2, mode=0)
    print("widths: terms at the edge of the range", flush=True)
    pl = binding.Planner(p, "cuda:0")
    pl.eval_cost_tables()
    pl.stage_dp()
    o, res = orc.Oracle(p), pl.results()
    per = o.n_orders() * 2
    seen = set()
    for k, cfg in enumerate(o.configs()):
        pairs = _overflows(o, 8, 3, cfg, range(1, 7))
        every = pairs or _overflows(o, 8, 3, cfg, [7])
        nominal = any(o.dp_const(cfg, order) >= 2 ** 44 for order in range(o.n_orders()))
        over = res["status"][k * per:(k + 1) * per] == 2
        assert over.all() == over.any() == (every or nominal), (cfg, every, nominal)
        seen.add((every, pairs or nominal))
    assert {(True, False), (False, False)} <= seen   # only the set of three; none at all


def _canonical_path(cost, flags, t):
    """The least-sum path at threshold t: from the last stage the smallest split point,
    then the smallest width.  (layers, widths, recomputation) of every stage."""
    big = np.int64(1) << 60
    pp, units, _, w1, _ = cost.shape
    f = np.full((pp + 1, units, w1), big)
    f[0, 0, 0] = 0
    for s in range(pp):
        for w in (1, 2, 3):
            for u in range(units - w):
                if f[s, u].min() < big:
                    c = cost[s, u, w - 1]
                    v = np.where(c <= t, np.minimum(f[s, u][:, None] + np.minimum(c, big), big), big).min(axis=0)
                    f[s + 1, u + w] = np.minimum(f[s + 1, u + w], v)
    b, u, path = w1 - 1, units - 1, []
    for s in range(pp - 1, -1, -1):
        a, w = next((a, w) for a in range(b) for w in (1, 2, 3)
                    if u >= w and f[s, u - w, a] < big and cost[s, u - w, w - 1, a, b] <= t
                    and f[s, u - w, a] + cost[s, u - w, w - 1, a, b] == f[s + 1, u, b])
        path.append((b - a, w, int(flags[s, u - w, w - 1, a, b]), u - w))
        b, u = a, u - w
    return path[::-1]


@pytest.mark.parametrize("counts", [[256, 256], [256, 128, 128]])
def test_partitions_of_the_last_tier(torch, counts):
    """100 layers, 16 stages, no windows: more keys with their lists in the workspace
    than it has slices, each with four groups of equal min(B, PP).  Layers, widths,
    stage types and recomputation against the canonical path on the oracle's costs, and
    the whole launch against launches of a few keys."""
    micro = [1, 5, 16, 40, 16]
    p = widths(workloads.random_tiny(61, n_layers=100, n_types=len(counts), max_pp=16, micro=micro), prune_window=0,
               allow_recompute=1)
    m, c = p["model"], p["cluster"]
    m.update(n_experts=8, top_k=2, hidden=512, seq_len=1024)
    m["expert_tokens"] = np.full((100, 8), 256, dtype=np.int64)
    m["is_moe"] = (np.arange(100) % 3 > 0).astype(np.uint8)
    c["count"] = np.array(counts, dtype=np.int32)
    c["mem_bytes"] = np.array([60, 90, 75][:len(counts)], dtype=np.int64) * 10**9
    p["space"].update(pp_max=16, tp_mask=15, cp_mask=15, tpe_mask=15, ep_max=8, mode=0)
    print(f"widths: last tier, devices {counts}", flush=True)
    pl = binding.Planner(p, "cuda:0")
    pl.eval_cost_tables()
    pl.stage_dp()
    in_ws = int(pl.d_dp_ws[4:8].cpu().numpy().view(np.uint32)[0])
    assert in_ws > 256
    res, types, wd = pl.results().copy(), pl.stage_types().copy(), pl.widths().copy()
    deep = np.nonzero(pl.cand_host["pp"] == 16)[0]
    first, n = int(deep[0]), len(deep)
    for x in (pl.d_res, pl.d_types, pl.d_widths):
        x[first * x.numel() // pl.n:].zero_()
    for at in range(first, first + n, 5 * 150):   # whole keys, at most 150 a launch
        pl.stage_dp(first=at, count=min(5 * 150, first + n - at))
    assert (pl.results() == res).all()
    assert (pl.stage_types() == types).all() and (pl.widths() == wd).all()

    o = orc.Oracle(p)
    per = o.n_orders() * len(micro)
    key = deep.reshape(-1, 5)
    ok = (res["status"][key] == 0).all(axis=1)
    mixed = (res["recompute_mask"][key[:, 2]] > 0) & ok   # recomputes somewhere
    keys = [key[np.nonzero(mixed)[0][0]], key[np.nonzero(mixed)[0][-1]]]
    recomputed = 0
    for i in [int(keys[0][0]), int(keys[0][1]), int(keys[0][2]), int(keys[0][3]), int(keys[1][2])]:
        cfg, order = o.configs()[i // per], i % per // len(micro)
        cost, flags = o.width_costs(i)
        b = int(pl.cand_host["n_micro"][i])
        obj, total, largest = _numpy_sweep(cost, b)
        path = _canonical_path(cost, flags, largest)
        got = res[i]
        assert (int(got["stage_sum"]), int(got["t_max"])) == (total, largest)
        assert int(got["objective"]) == obj + o.dp_const(cfg, order)
        assert got["layers"][:16].tolist() == [x[0] for x in path] and wd[i][:16].tolist() == [x[1] for x in path]
        assert [(int(got["recompute_mask"]) >> s) & 1 for s in range(16)] == [x[2] for x in path]
        assert types[i][:16].tolist() == [o.width_stage(cfg, order, s, x[3], x[1], b)["mask"] for s, x in enumerate(path)]
        recomputed += sum(x[2] for x in path)
    same = key[ok]   # the two candidates with B = 16
    assert (res[same[:, 2]] == res[same[:, 4]]).all() and recomputed > 0
