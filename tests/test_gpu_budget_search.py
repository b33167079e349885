"""Budget search at the edges of its kernel: scores that just fit and just exceed the LDS cache, one unit of a kind, layers
that no wave or block divides, units that cost nothing."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_parity import _budget_check, _gate_case, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nl,Hq,Hk,F,zero", [(64, 4, 2, 512, None), (3, 12, 4, 10923, None), (1, 1, 1, 1, None), (17, 64, 64, 65, None),
                                             (5, 8, 2, 1025, "ffn"), (5, 8, 2, 1025, "head")])
def test_budget_search_edges(nl, Hq, Hk, F, zero):
    _say(f"budget_search nl={nl} Hq={Hq} Hk={Hk} F={F} zero={zero}")
    desc, gh, gf, gh_h, gf_h, P = _gate_case(nl, 2, Hq, Hk, F, 16, 0, seed=nl + F)
    rng = np.random.default_rng(F)
    costs = [rng.integers(1000, 5000, nl).tolist(), rng.integers(500, 2000, nl).tolist(), rng.integers(5, 40, nl).tolist()]
    if zero:
        costs[2 if zero == "ffn" else 0] = [0] * nl
    dense = sum(Hq * costs[0][l] + Hk * costs[1][l] + F * costs[2][l] for l in range(nl))
    floor = sum(costs[0][l] + costs[1][l] + costs[2][l] for l in range(nl))
    for budget in (dense, dense - 1, int(0.6 * dense), int(0.1 * dense), floor, floor - 1):
        _budget_check(desc, gh, gf, gh_h, gf_h, P - 1, Hk, tuple(costs), 0, budget)
