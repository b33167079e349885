"""Budget search at the edges of its kernel: scores that just fit and just exceed the LDS cache, one unit of a kind, layers
that no wave or block divides, units that cost nothing."""
from __future__ import annotations

import numpy as np
import pytest
import torch

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


# Scores that leave the histogram of equal steps: all equal, two values (more units in a step than its list holds), an outlier
# that puts the others into one step, an infinity, a layer that has only zeros, and a range too narrow for steps.  The last model's
# groups and channels fit the kernel's LDS, its heads do not
@pytest.mark.parametrize("kind", ["equal", "two", "outlier", "inf", "zeros", "narrow"])
@pytest.mark.parametrize("nl,Hq,Hk,F", [(3, 8, 4, 700), (20, 4, 2, 130), (2, 4, 2, 19000), (64, 64, 64, 512)])
def test_budget_search_degenerate_scores(nl, Hq, Hk, F, kind):
    _say(f"budget_search nl={nl} F={F} {kind}")
    desc, gh, gf, gh_h, gf_h, P = _gate_case(nl, 2, Hq, Hk, F, 16, 0, seed=nl + F)
    gh_h, gf_h = np.array(gh_h), np.array(gf_h)
    for a in (gh_h, gf_h):
        if kind == "equal":
            a[:] = 0.5
        elif kind == "two":
            a[:] = np.where(a < np.median(a), 0.25, 0.75)
        elif kind == "outlier":
            a.reshape(-1)[a.size // 2] = 3e30
        elif kind == "inf":
            a.reshape(-1)[a.size // 2] = np.inf
        elif kind == "narrow":
            a *= np.float32(1e-37)
        else:
            a[0] = 0.0
    gh.copy_(torch.from_numpy(gh_h).reshape(gh.shape))
    gf.copy_(torch.from_numpy(gf_h).reshape(gf.shape))
    rng = np.random.default_rng(F)
    costs = [rng.integers(1000, 5000, nl).tolist(), rng.integers(500, 2000, nl).tolist(), rng.integers(5, 40, nl).tolist()]
    dense = sum(Hq * costs[0][l] + Hk * costs[1][l] + F * costs[2][l] for l in range(nl))
    floor = sum(costs[0][l] + costs[1][l] + costs[2][l] for l in range(nl))
    for budget in (dense, dense - 1, int(0.6 * dense), int(0.1 * dense), floor):
        _budget_check(desc, gh, gf, gh_h, gf_h, P - 1, Hk, tuple(costs), 0, budget)
