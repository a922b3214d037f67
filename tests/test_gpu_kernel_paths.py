"""GPU parity of single paths of the kernels at the sizes where each can go wrong
(edges of its range, remainders, the largest values), against the oracle.

Every quantity is an integer and must match exactly.
"""
import numpy as np
import pytest

import oracle
from oracle import ALPHA_INF
from test_gpu_simulate import assert_same, dev, gpu_sim, log  # noqa: F401  (dev: the fixture)

pytestmark = pytest.mark.gpu


def check(dev, ctx, a, p, o, prefill=False, **kw):
    log(ctx)
    got, gs, gf = gpu_sim(dev, a, p, o, prefill=prefill, **kw)
    ref, rs, rf = oracle.simulate(a, p, o, schedule=True,
                                  flags=oracle.FLAG_PREFILL if prefill else 0, **kw)
    assert_same(ctx, got, ref, gs, rs, gf, rf)
    return got


@pytest.mark.parametrize("policy,n,B,alpha,M_kv,prefill", [
    ("fcfs", 1000, 1000, ALPHA_INF, 0, False),
    ("isjl", 1000, 1000, ALPHA_INF, 1 << 40, False),  # a budget that no 32-bit sum reaches
    ("ljf", 1000, 1000, 5, (1 << 31) + 7, False),
    ("isjl", 500, 500, 1 << 10, (1 << 29) + 12345, False),
    ("sjf", 120, 100, ALPHA_INF, (1 << 26), False),
    ("fcfs", 1000, 1000, ALPHA_INF, (1 << 29) + 77, True),
    ("isjl", 130, 128, 2, 1 << 33, True),
])
def test_largest_reservations_and_footprints(dev, policy, n, B, alpha, M_kv, prefill):
    """Jobs just below 2^20 tokens on up to 1,000 workers: reservations and footprint
    sums near 2^30, the range that the 32-bit span sums are exact over."""
    rng = np.random.default_rng(n + B)
    size = (2, n)
    a = np.sort(rng.integers(0, 40, size=size), axis=1).astype(np.int32)
    if prefill:
        o = rng.integers(1, 60, size=size).astype(np.int32)
        p = ((1 << 20) - 1 - o - rng.integers(0, 300, size=size)).astype(np.int32)
    else:
        o = rng.integers(1, 3000, size=size).astype(np.int32)
        p = ((1 << 20) - 1 - o - rng.integers(0, 3, size=size)).astype(np.int32)
        p[1] = p[1] // 64  # a shorter instance beside it, where the starts spread further
    check(dev, f"{policy} n={n} B={B} M={M_kv} prefill={prefill}", a, p, o, prefill=prefill,
          policy=policy, B=B, alpha=alpha, M_kv=M_kv, cost_c=3, cost_tau=2)
