"""Test-side helpers of the GPU parity tests: the margin rule for a floating-point top-U
decision, and the LayerNorm launch to the bit.  (The device plumbing lives in paper_2604_08971_amd.device_model.)"""
from __future__ import annotations

from typing import Optional

import numpy as np

from paper_2604_08971_amd import workloads as W
from paper_2604_08971_amd.device_model import (ORACLE_MODE, SF_DTYPE, DeviceModel, desc_for,  # noqa: F401
                                               key_valid_host, to_dev, to_host)


def selection_report(score_oracle: np.ndarray, sel_gpu: np.ndarray, sel_oracle: np.ndarray,
                     valid: Optional[np.ndarray], eps_rel: float):
    """Margin check of one (sample, head): the GPU's active set is acceptable iff
    every chosen query scores >= tau - eps and every allowed query left out
    scores <= tau + eps, tau being the oracle's U-th largest score.
    Returns (ok, differs)."""
    L = score_oracle.shape[0]
    chosen = sel_gpu[sel_gpu >= 0]
    ref = sel_oracle[sel_oracle >= 0]
    if len(chosen) != len(ref) or len(np.unique(chosen)) != len(chosen):
        return False, True
    if len(ref) == 0:
        return True, False
    if not np.all(np.diff(chosen) > 0):
        return False, True
    allowed = np.ones(L, bool) if valid is None else valid.astype(bool)
    if not allowed[chosen].all():
        return False, True
    tau = np.min(score_oracle[ref])
    eps = eps_rel * max(1.0, abs(tau))
    mask = np.zeros(L, bool)
    mask[chosen] = True
    ok = bool(np.all(score_oracle[chosen] >= tau - eps) and
              np.all(score_oracle[allowed & ~mask] <= tau + eps))
    return ok, not np.array_equal(chosen, ref)


def _fma32(a, b, c):
    """float32 a * b + c rounded once (the float64 sum of the exact product is rounded first: it matters once in 2^29)."""
    return (a.astype(np.float64) * b + c).astype(np.float32)


def layernorm_as_launched(x: np.ndarray, gamma: np.ndarray, beta: np.ndarray, half: str, eps: float = 1e-5) -> np.ndarray:
    """The library's LayerNorm launch of 16-bit rows (d % 8 == 0) to the bit, from 16-bit values: lane l of a wave adds columns 8 l .. 8 l + 7
    of every 512 one after the other, lanes 32, 16, .. 1 apart are joined, and the last product rounds to 16 bits by itself
    in binary16."""
    rows, d = x.shape
    nch = -(-d // 512)
    v = np.zeros((rows, nch * 512), np.float32)
    v[:, :d] = x
    inside = np.zeros(nch * 512, bool)
    inside[:d] = True
    v, inside = v.reshape(rows, nch, 64, 8), inside.reshape(nch, 64, 8)

    def joined(s):
        for o in (32, 16, 8, 4, 2, 1):
            s = s + s[:, np.arange(64) ^ o]
        return s[:, :1]

    s = np.zeros((rows, 64), np.float32)
    for c in range(nch):
        for e in range(8):
            s = s + v[:, c, :, e]
    mean = joined(s) / np.float32(d)
    t = np.where(inside, v - mean[:, :, None, None], np.float32(0))
    q = t[:, 0, :, 1] * t[:, 0, :, 1]
    for c in range(nch):
        for e in range(8):
            if (c, e) != (0, 1):
                q = _fma32(t[:, c, :, e], t[:, c, :, e], q)
    inv = np.float32(1) / np.sqrt(joined(q) / np.float32(d) + np.float32(eps))
    n = ((v - mean[:, :, None, None]) * inv[:, :, None, None]).reshape(rows, -1)[:, :d]
    if half == "f16":
        return (n.astype(np.float64) * gamma + beta).astype(np.float16).astype(np.float32)
    return W.to_bf16_values(_fma32(n, gamma, beta))
