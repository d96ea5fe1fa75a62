"""The launch rules that depend on a call's size: the arg-min over few candidates in
one launch, the stage DP with one workgroup a key, the 1F1B walk with four waves a
SIMD, at and around their limits."""
import copy

import numpy as np
import pytest

from paper_2609_39350_amd import binding, workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def planner():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = copy.deepcopy(workloads.config(2))
    p["space"]["micro"] = [8]   # six candidates a configuration
    pl = binding.Planner(p, "cuda:0")
    pl.run()
    return pl


def check_arg_min(pl, per, n, batch):
    """Least (objective, index) of the first n records and of every configuration's,
    against numpy on the same records; with a fixed global batch only some count."""
    problem = copy.deepcopy(pl.problem)
    problem["space"]["global_batch"] = batch
    res, cand = pl.results()[:n], pl.cand_host[:n]
    take = res["status"] == 0
    if batch:
        take &= cand["n_micro"].astype(np.int64) * cand["dp"] * problem["model"]["micro_batch_size"] == batch
    obj = np.where(take, res["objective"], np.iinfo(np.int64).max)
    pl.d_config_best.fill_(-7)
    try:
        plan = binding.best_plan(problem, pl.d_cand, pl.d_tables, pl.d_res, n, pl.d_ws, pl.d_config_best)
        assert take.any() and plan["instance"] == int(np.argmin(obj)) and plan["objective"] == int(obj.min())
    except binding.HapmoeError as e:
        assert e.code == -6 and not take.any()
    got = pl.config_best()
    for c in range(pl.n_configs):
        seg = obj[c * per:(c + 1) * per]
        want = -1 if len(seg) == 0 or seg.min() == np.iinfo(np.int64).max else c * per + int(np.argmin(seg))
        assert got[c] == want, (c, int(got[c]), want)


@pytest.mark.parametrize("n", [1, 5, 6, 7, 2047, 2048, 2049, 5424])
@pytest.mark.parametrize("batch", [0, 32])
def test_arg_min_around_the_one_launch_limit(planner, n, batch):
    print(f"arg-min of {n} records, batch {batch}", flush=True)
    check_arg_min(planner, 6, n, batch)


@pytest.mark.parametrize("orders,counts", [(2, 8), (2, 9), (6, 2), (6, 3)])   # one launch up to 16 a configuration
@pytest.mark.parametrize("n", [11, 13, 2047, 2048, 2049, 4000])
def test_arg_min_of_long_segments(planner, orders, counts, n):
    p = copy.deepcopy(planner.problem)
    if orders == 2:   # two device types
        c = p["cluster"]
        c["n_types"] = 2
        for f in ("count", "speed", "mem_bytes", "eff", "route_coef", "t_dense", "t_ffn"):
            c[f] = c[f][:2]
        c["bw"], c["alpha"], c["count"] = c["bw"][:2, :2], c["alpha"][:2, :2], np.array([32, 32], dtype=np.int32)
    p["space"]["micro"] = [8, 16, 32, 64, 128, 5, 6, 7, 9][:counts]
    pl = binding.Planner(p, "cuda:0")
    pl.run()
    print(f"arg-min of {n} records, {orders * counts} a configuration", flush=True)
    check_arg_min(pl, orders * counts, n, 0)


@pytest.mark.parametrize("layers,experts", [(32, 64), (33, 64), (31, 66), (64, 32), (127, 16), (8, 256), (8, 257), (9, 0)])
def test_load_imbalance_factors_of_either_kernel(planner, layers, experts):
    """1 + gamma (rho - 1) of every layer, reduced by the cost-table workgroups (up to
    2,048 counts) or by a kernel before them."""
    e = max(experts, 1)
    p = workloads.random_tiny(40 + layers, n_layers=layers, n_types=2)
    rng = np.random.default_rng(layers * 1000 + experts)
    p["model"].update(n_experts=experts, top_k=1)
    p["model"]["is_moe"] = (rng.random(layers) < 0.8).astype(np.uint8) * (experts > 0)
    p["model"]["params_expert"] = np.where(p["model"]["is_moe"], 10**6, 0).astype(np.int64)
    tokens = rng.integers(0, 1000, size=(layers, e)).astype(np.int64)
    p["model"]["expert_tokens"] = tokens if experts else np.zeros((layers, 0), dtype=np.int64)
    p["params"]["gamma"] = 0.5
    print(f"load imbalance, {layers} layers x {experts} experts", flush=True)
    pl = binding.Planner(p, "cuda:0")
    pl.eval_cost_tables()
    layout = binding.tables_layout(p)
    at = -(-(layout["off_time"] + layout["n_configs"] * layout["n_masks"] * 3 * layout["np"] * 8) // 256) * 256
    got = pl.tables()[at:at + 8 * layers].view(np.float64)
    rho = (tokens.max(axis=1) * e).astype(np.float64) / tokens.sum(axis=1).astype(np.float64)
    want = np.where(p["model"]["is_moe"], 1.0 + 0.5 * (rho - 1.0), 1.0)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("objective", ["threshold", "1f1b"])
def test_stage_dp_one_workgroup_a_key(planner, objective):
    """Sub-ranges with fewer keys than resident workgroups (no work queue) give the
    records of the whole launch, which has more."""
    pl = planner
    pl.stage_dp(objective=objective)
    whole = pl.results().copy()
    pl.d_res.zero_()
    print(f"stage DP in sub-ranges, {objective}", flush=True)
    cuts = [0, 1, 64, 65, 1000, 2500, 3999, pl.n]
    for a, b in zip(cuts[:-1], cuts[1:]):
        pl.stage_dp(first=a, count=b - a, objective=objective)
    assert (pl.results() == whole).all()
    pl.stage_dp()


@pytest.mark.parametrize("window,least", [(1, 24576), (0, 32768)])
def test_1f1b_four_waves_a_simd(planner, window, least):
    """At least `least` keys run the walk built for four waves a SIMD, fewer the other
    one: both give the same records and statistics (39,264 keys of three counts)."""
    p = copy.deepcopy(workloads.config(3))
    p["params"]["prune_window"] = window
    pl = binding.Planner(p, "cuda:0")
    pl.eval_cost_tables()
    print(f"1F1B walk, 39,264 keys, windows {window}", flush=True)
    pl.stage_dp(objective="1f1b", stats=True)
    whole, stats = pl.results().copy(), pl.stats().copy()
    assert (whole["status"] == 0).sum() > 1000
    cuts = [0, 3 * (least - 1), pl.n] if window else [0, 3 * 7000, 3 * (least + 6000), pl.n]
    for with_stats in (False, True):
        pl.d_res.zero_()
        for a, b in zip(cuts[:-1], cuts[1:]):
            pl.stage_dp(first=a, count=b - a, objective="1f1b", stats=with_stats)
            if with_stats:
                assert (pl.stats()[a:b] == stats[a:b]).all()
        assert (pl.results() == whole).all()


@pytest.mark.parametrize("objective", ["threshold", "1f1b"])
def test_work_queue_and_a_workgroup_a_key(planner, objective):
    """60,240 keys of 64 counts, up to 32 stages, go through the work queue; a few
    thousand of them, the deepest, the shallowest and some between, one workgroup each."""
    p = copy.deepcopy(workloads.config(4))
    pl = binding.Planner(p, "cuda:0")
    pl.eval_cost_tables()
    print(f"stage DP, 60,240 keys and 2,000, {objective}", flush=True)
    pl.stage_dp(objective=objective)
    whole = pl.results().copy()
    assert (whole["status"] == 0).sum() > 10**6
    for first, count in ((0, 128000), (1900003, 128001), (pl.n - 128000, 128000)):
        pl.d_res.zero_()
        pl.stage_dp(first=first, count=count, objective=objective)
        part = pl.results()
        assert (part[first:first + count] == whole[first:first + count]).all()
        assert not part[:first]["layers"].any() and not part[first + count:]["layers"].any()
