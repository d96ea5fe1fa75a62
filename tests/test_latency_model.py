"""The model of the least-latency range search (tests/latency_model.py) against the
oracle's threshold sweep on explicit cost tensors: every member's least latency and
its largest stage."""
import numpy as np
import pytest

from oracle import oracle as orc
from tests.latency_model import Search


@pytest.mark.parametrize("seed", range(12))
def test_model_equals_threshold_sweep(seed):
    rng = np.random.default_rng(seed)
    n, pp = int(rng.integers(6, 18)), int(rng.integers(2, 6))
    times = rng.integers(1, (40, 10**6, 10**12)[seed % 3], size=n)   # ties, 32-bit and 64-bit costs
    ends = np.concatenate([[0], np.cumsum(times)])
    slow = rng.integers(1, 4, size=pp)
    lo, hi = [1] * pp, [n - pp + 1] * pp
    cost = np.full((pp, n + 1, n + 1), orc.INF, dtype=np.int64)
    for a in range(n):
        for b in range(a + 1, n + 1):
            cost[:, a, b] = (ends[b] - ends[a]) * slow
    micro = [pp + 1, pp + 1, pp + 3, pp + 20, 1000]
    best, passes, _ = Search(cost, lo, hi, micro).run()
    for b, (latency, largest) in zip(micro, best):
        ref = orc.dp_latency(pp, n, b, cost)
        largest = 3 * (largest >> 2) + (((largest & 3) + 1) >> 1)
        assert (latency, largest) == (ref["opt"], ref["tmax"])
    assert passes > 0
