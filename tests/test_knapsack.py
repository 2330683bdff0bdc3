"""The retrieval knapsack against the oracle's, where its parts meet: instances that the reduction decides
almost whole, instances in which nearly everything ties and nothing can be fixed, groups without tokens,
lengths with a common divisor, and values so large that the programme counts in 128 bits."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2510_18546_amd import binding as B


def instance(kind, rng):
    n = int(rng.integers(17, 90))
    lens = rng.integers(0, 70, n)
    if kind == "spread":
        p = rng.standard_normal(n)
    elif kind == "tied":                       # few distinct scores, one length: many optimal sets
        lens, p = np.full(n, 5), rng.integers(1, 3, n) / 4
    elif kind == "equal ratio":                # value per token nearly the same: the relaxation fixes little
        p = lens * 0.0078125 + rng.integers(0, 2, n) * 2.0 ** -20
    elif kind == "divisor":                    # around a multiple of 64 columns once divided
        lens, p = rng.integers(1, 9, n) * 24, rng.standard_normal(n)
    elif kind == "large values":
        p = rng.standard_normal(n) * 2.0 ** 20
    return lens.astype(np.int32), p.astype(np.float32)


@pytest.mark.parametrize("kind", ["spread", "tied", "equal ratio", "divisor", "large values"])
def test_knapsack_matches_oracle(oracle, kind):
    rng = np.random.default_rng(len(kind))
    for _ in range(25):
        lens, p = instance(kind, rng)
        pool = B.kv_pool_create(None, None, lens, n_q_heads=4, rope_base=1e4, max_ctx=1 << 20, dtype=B.EN_BF16,
                                k_ptr=0x1000, v_ptr=0x2000, shape=(len(lens), 1, max(1, int(lens.max())), 64))
        for budget in {0, 1, 63, 64, int(lens.sum()) // 3, int(rng.integers(0, lens.sum() + 2)), int(lens.sum()) - 1}:
            got = B.segment_select_scored(pool, p, 0.0, max(budget, 0), 1, want_plan=False)[0].tolist()
            assert got == oracle.knapsack_dp(p, lens, 0.0, max(budget, 0)), (kind, budget)


def test_knapsack_stays_within_its_bound():
    """Long candidates with values that count in 128 bits, just accepted (the bound is 1 GiB): the call takes no more
    than the bound."""
    code = """
import itertools, resource
import numpy as np
from paper_2510_18546_amd import binding as B
lens, p, budget = np.array([19999999, 20000003, 20000017], np.int32), np.array([1.5, 1.0, 1.25], np.float32) * 2.0 ** 20, 40000018
pool = B.kv_pool_create(None, None, lens, n_q_heads=4, rope_base=1e4, max_ctx=1 << 20, dtype=B.EN_BF16, k_ptr=0x1000,
                        v_ptr=0x2000, shape=(3, 1, int(lens.max()), 64))
B.segment_select_scored(pool, p, 0.0, 1, 1, want_plan=False)
before = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss
got = B.segment_select_scored(pool, p, 0.0, budget, 1, want_plan=False)[0].tolist()
sets = [s for n in range(4) for s in itertools.combinations(range(3), n) if sum(int(lens[g]) for g in s) <= budget]
assert got == list(max(sets, key=lambda s: sum(float(p[g]) for g in s))), got
grown = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss - before
assert grown <= 1 << 20, grown
"""
    subprocess.run([sys.executable, "-c", code], check=True, cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
