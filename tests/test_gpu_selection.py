"""The k largest of a row - active queries, keep sets - where the values are degenerate: equal, two of them, an outlier that leaves
the others in one step of the histogram, infinities."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2604_08971_amd import binding as sf
from test_gpu_parity import _say

pytestmark = pytest.mark.gpu


def _expected(score, allowed, U):
    """Highest scores first, ties to the lower index, ascending."""
    key = np.where(allowed, score, -np.inf)
    order = np.lexsort((np.arange(len(key)), -key))[:min(U, int(allowed.sum()))]
    return np.sort(order)


# The selection against the device's own scores: all equal (a range of one value), two values, an outlier that leaves the others
# in one step of the histogram, an infinity.  One to four queries per thread
# in registers, and more of them read from LDS, in the one launch of a short sequence (300 and 700 keys) and in one of their own.
@pytest.mark.parametrize("dtype,L,dh", [("bf16", 300, 64), ("bf16", 700, 32), ("bf16", 200, 128), ("bf16", 300, 128), ("bf16", 3000, 64), ("bf16", 5000, 128), ("f32", 90, 16), ("f32", 700, 16)])
@pytest.mark.parametrize("kind", ["equal", "two", "outlier", "inf", "random"])
def test_selection_of_degenerate_scores(dtype, L, dh, kind):
    _say(f"selection {dtype} L={L} {kind}")
    B, nH, U = 2, 3, 37
    rng = np.random.default_rng(L)
    Q, K, V = (rng.standard_normal((B, nH, L, dh)).astype(np.float32) for _ in range(3))
    if kind in ("equal", "two"):
        Q[:] = 0
        if kind == "two":
            Q[:, :, rng.choice(L, L // 2, replace=False), 0] = 1.0
    elif kind == "outlier":
        Q[:, :, L // 3] *= 1e4
    elif kind == "inf":
        Q[:, :, L // 3] = 0
        Q[:, :, L // 3, 0], K[:, :, 5, 0] = -1e30, 1e16
    kv = (rng.random((B, L)) < 0.8).astype(np.uint8)
    kv[:, [5, L // 3]] = 1
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    desc = sf.make_desc(B, L, 64, nH, nH, dh, 64, dtype=sf.SF_F32 if dtype == "f32" else sf.SF_BF16, U_override=U)
    _, sel, score = sf.sparse_gqa_forward(desc, *(torch.from_numpy(x).cuda().to(td) for x in (Q, K, V)),
                                          torch.arange(nH, dtype=torch.int32, device="cuda").reshape(1, nH),
                                          key_valid=torch.from_numpy(kv).cuda(), want_score=True)
    torch.cuda.synchronize()
    sel, score = sel.cpu().numpy(), score.cpu().numpy()
    if kind == "equal":
        assert (score[:, :, kv[0] == 1][0] == 0).all()
    if kind == "inf":
        assert np.isposinf(score[:, :, L // 3]).all()
    for b in range(B):
        for h in range(nH):
            assert not np.isnan(score[b, h]).any()
            assert np.array_equal(sel[b, h], _expected(score[b, h], kv[b].astype(bool), U)), (b, h)


@pytest.mark.parametrize("F", [1, 63, 700, 1024, 4096, 4097, 16384])
@pytest.mark.parametrize("kind", ["random", "equal", "two", "outlier", "inf", "narrow"])
def test_keep_masks_of_degenerate_scores(F, kind):
    _say(f"keep masks F={F} {kind}")
    rng = np.random.default_rng(F)
    g = rng.random((2, 1, F)).astype(np.float32)
    if kind == "equal":
        g[:] = 0.25
    elif kind == "two":
        g = np.where(g < 0.7, np.float32(0.5), np.float32(-0.0))
    elif kind == "outlier":
        g[:, :, F // 2] = 3e38
    elif kind == "inf":
        g[0, :, F // 2], g[1, :, F // 3] = np.inf, -np.inf
    elif kind == "narrow":                       # ranges too narrow for steps: below the normal numbers, and of normal ones
        g[0] *= np.float32(1e-38)
        g[1] *= np.float32(1e-31)
    desc = sf.make_desc(1, 64, 64, 4, 2, 16, F, n_layers=2, dtype=sf.SF_F32)
    for k in {1, max(1, F // 2), F}:
        m = sf.gate_scores_to_masks(desc, torch.rand((2, 1, 4), device="cuda"), torch.from_numpy(g).cuda(), [1, 1], [k, k])
        torch.cuda.synchronize()
        idx, mask = m["ffn_idx"].cpu().numpy().reshape(2, F), m["ffn_mask"].cpu().numpy().reshape(2, F)
        for l in range(2):
            want = _expected(g[l, 0], np.ones(F, bool), k)
            assert np.array_equal(idx[l, :k], want) and (idx[l, k:] == -1).all()
            assert np.array_equal(np.flatnonzero(mask[l]), want)
