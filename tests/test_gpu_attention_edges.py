"""SentryAttend at the edges of its dispatch: key ranges of the score stream and of the statistics, keys dealt to waves, one
and two query blocks per wave, head dimension 128, the fill beside the selection, masks that leave whole tiles out."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import cpu_oracle as orc
from oracle.packs import err_metric
from paper_2604_08971_amd import binding as sf
from paper_2604_08971_amd import workloads as W
from gpu_utils import SF_DTYPE, to_dev, to_host
from helpers import make_wl
from test_gpu_tokens_packed import _packed_case
from test_gpu_parity import TOL, _encoder_parity, _gqa_case, _say, test_sparse_gqa_parity as gqa_case

pytestmark = pytest.mark.gpu


# B, heads, groups, length, head dim, U override, mask
@pytest.mark.parametrize("dtype,B,nH,nG,L,dh,Uo,mask", [
    ("bf16", 1, 6, 2, 33, 64, -1, True),          # two tiles, the second of one key
    ("bf16", 1, 1, 1, 1025, 32, -1, False),       # statistics in two launches, score parts, last tile of one key
    ("bf16", 2, 3, 1, 2047, 64, 33, True),        # one active query beyond a block
    ("bf16", 130, 2, 2, 97, 64, 33, True),        # two query blocks per wave, four waves
    ("bf16", 130, 2, 1, 97, 32, 64, False),
    ("bf16", 3, 5, 5, 515, 128, 40, True),        # head dimension 128
    ("bf16", 2, 2, 1, 700, 128, 255, False),      # just below the staged kernels
    ("bf16", 2, 2, 1, 700, 128, 256, True),       # and just there
    ("bf16", 1, 64, 8, 64, 32, 0, False),         # no active query: every row is filled
    ("f32", 2, 3, 1, 17, 4, 3, True),             # fp32: one query past a block, the narrowest head
    ("f32", 1, 2, 2, 31, 96, 30, True),           # one key short of a tile, a head between one and two waves
    ("f32", 1, 4, 2, 65, 256, 64, False),         # one key past two tiles, the widest head
])
def test_attention_edges(dtype, B, nH, nG, L, dh, Uo, mask):
    gqa_case(dtype, B, nH, nG, L, dh, Uo, mask)


# Which of the two kernels takes fewer than 256 active rows is an estimate of their times: the plan is asserted, so that every
# form stays covered (by the second of two calls, with an output that is not aligned, where one launch serves the first).  Staged tiles: key splits with key groups inside a workgroup, four waves, a group with more pairs than
# waves, each head dimension; sliced keys: four waves with one query block each.
@pytest.mark.parametrize("B,nH,nG,L,dh,Uo,mask,staged,splits", [
    (1, 2, 1, 4097, 64, -1, True, 1, 13),         # last tile of one key
    (3, 3, 1, 9000, 32, -1, False, 1, 29),
    (2, 2, 1, 2049, 128, -1, True, 1, 7),
    (130, 4, 2, 97, 64, 33, True, 1, 1),          # four waves
    (130, 10, 2, 97, 64, 64, False, 1, 1),        # ten pairs
    (130, 8, 2, 97, 32, 33, True, 1, 1),
    (130, 2, 2, 97, 128, 33, False, 1, 1),
    (130, 4, 4, 97, 64, 31, True, 0, 1),
    (130, 4, 4, 65, 128, 32, True, 0, 1),
    (130, 6, 2, 65, 32, 32, False, 0, 1),
])
def test_active_pass_kernels(B, nH, nG, L, dh, Uo, mask, staged, splits):
    plan = sf.sparse_gqa_plan(sf.make_desc(B, L, 64, 8, 2, dh, 64, dtype=sf.SF_BF16, U_override=Uo), nH, nG)
    assert (plan["staged"], plan["splits"]) == (staged, splits), plan
    gqa_case("bf16", B, nH, nG, L, dh, Uo, mask)


# Rows of few heads that are filled by many blocks (256 KB a head, half of it with a caller's list; the last block's rows end
# with the sequence): every row that is not active is its group's context vector
@pytest.mark.parametrize("dtype,B,nH,nG,L,dh,forced", [
    ("bf16", 1, 3, 1, 2049, 64, False), ("bf16", 2, 2, 2, 4097, 32, False), ("bf16", 1, 2, 1, 1031, 128, True),
    ("f32", 1, 2, 1, 1025, 64, False), ("f32", 2, 1, 1, 601, 96, True),
])
def test_rows_of_few_heads(dtype, B, nH, nG, L, dh, forced):
    _say(f"few heads {dtype} B={B} nH={nH} L={L} dh={dh} forced={forced}")
    _gqa_case(dtype, B, nH, nG, L, dh, -1, True, seed=L, forced=forced)


def test_packed_rows_of_few_heads():
    _say("few heads, packed")
    _packed_case(make_wl(W.small_spec(dtype="bf16", d=64, Hq=2, Hk=1, dh=32, F=128, nl=1, seg=(2900, 1300), B=2, head_keep=1.0, dropout="upto:1")))


# one sample whose only modality is a few tokens at the end: most key tiles are dead; a length that one launch serves, and one
# that keeps the separate ones
@pytest.mark.parametrize("seg", [(600, 40, 7), (1300, 80, 7)])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_encoder_with_dead_tiles(dtype, seg):
    _say(f"dead tiles {dtype} {seg}")
    spec = W.small_spec(dtype=dtype, B=7, seg=seg, d=64, Hq=2, Hk=1, dh=32, F=128, nl=1, head_keep=1.0,
                        dropout="upto:2", c=3)
    with sf.use_half("f16" if dtype == "f16" else "bf16"):
        _encoder_parity(make_wl(spec))


def test_forced_rows_behind_a_block_without_any():
    """A caller's list whose first 32 entries name no row (-1, or out of range, which counts as -1): the rows behind them are
    active rows like any other.  130 x 2 heads and 64 slots: two query blocks per wave."""
    B, nH, L, dh, U = 130, 2, 97, 32, 64
    rng = np.random.default_rng(5)
    Q, K, V = (W.to_bf16_values(rng.standard_normal(s).astype(np.float32)) for s in ((B, nH, L, dh), (B, 1, L, dh), (B, 1, L, dh)))
    fs = np.full((B, nH, U), -1, np.int32)
    fs[::2, :, :32] = L
    fs[:, :, 32:35] = [3, 40, L - 1]
    desc = sf.make_desc(B, L, 64, nH, 1, dh, 64, dtype=sf.SF_BF16, U_override=U)
    O = torch.full((B, L, nH * dh), float("nan"), dtype=torch.bfloat16, device="cuda")
    sf.sparse_gqa_forward_static(desc, *(to_dev(x, "bf16") for x in (Q, K, V)), torch.zeros((1, nH), dtype=torch.int32, device="cuda"),
                                 O, forced_sel=to_dev(fs, "bf16"))
    torch.cuda.synchronize()
    O = to_host(O)
    assert np.isfinite(O).all()
    O_ref, _, _, _ = orc.sparse_gqa(Q, K, V, np.zeros(nH, np.int32), U, None, np.where(fs < L, fs, -1).astype(np.int32), True, None)
    assert err_metric(O, O_ref) <= TOL["bf16"]


def test_allowed_query_whose_score_has_every_bit_set():
    """A query of NaNs with every bit set (memory filled with 0xff; of either sign, since the score subtracts) can score the NaN
    that maps to the smallest of all keys; it is still one of the allowed queries, and with no more of them than U the list
    names each of them."""
    B, nH, L, dh, U = 2, 2, 48, 16, 6
    rng = np.random.default_rng(6)
    Q, K, V = (rng.standard_normal((B, nH, L, dh)).astype(np.float32) for _ in range(3))
    kv = np.zeros((B, L), np.uint8)
    allowed = [5, 17, 30, 47]
    kv[:, allowed] = 1
    Q.view(np.uint32)[0, :, 17], Q.view(np.uint32)[1, :, 17] = 0xffffffff, 0x7fffffff
    desc = sf.make_desc(B, L, 64, nH, nH, dh, 64, dtype=sf.SF_F32, U_override=U)
    O, sel, _ = sf.sparse_gqa_forward(desc, *(torch.from_numpy(x).cuda() for x in (Q, K, V)),
                                      torch.arange(nH, dtype=torch.int32, device="cuda").reshape(1, nH), key_valid=torch.from_numpy(kv).cuda())
    torch.cuda.synchronize()
    assert (to_host(sel) == np.array(allowed + [-1] * (U - len(allowed)))).all()
    O = to_host(O).reshape(B, L, nH, dh)
    assert np.isfinite(np.delete(O, 17, axis=1)).all()


def test_score_over_key_ranges_keeps_nan_and_infinities():
    """The score of one sample comes in ranges of keys, the same sample in a batch of 64 without: NaN, both infinities and
    finite values fall on the same queries (one range has no allowed key, one key overflows its products)."""
    B, nH, L, dh = 64, 2, 600, 128
    rng = np.random.default_rng(8)
    Q, K, V = (W.to_bf16_values(rng.standard_normal((1, nH, L, dh)).astype(np.float32)) for _ in range(3))
    K[0, :, 350, 0] = 3e38
    Q[0, :, 100, 3] = np.nan
    Q[0, :, 102:104] = 0
    Q[0, :, 102, 0], Q[0, :, 103, 0] = 3e38, -3e38
    kv = np.ones((1, L), np.uint8)
    kv[0, 128:256] = 0
    hg = torch.arange(nH, dtype=torch.int32, device="cuda").reshape(1, nH)
    got = []
    for n in (1, B):
        desc = sf.make_desc(n, L, 64, nH, nH, dh, 64, dtype=sf.SF_BF16)
        parts = sf.sparse_gqa_plan(desc, nH, nH)["score_parts"]
        assert parts > 1 if n == 1 else parts == 1, parts
        q, k, v = (to_dev(np.repeat(x, n, axis=0), "bf16") for x in (Q, K, V))
        _, sel, score = sf.sparse_gqa_forward(desc, q, k, v, hg, key_valid=torch.from_numpy(np.repeat(kv, n, axis=0)).cuda(), want_score=True)
        torch.cuda.synchronize()
        got.append((to_host(sel)[0], to_host(score)[0]))
    (sel, score), (sel_ref, ref) = got
    assert np.isnan(ref[:, [100, 102]]).all() and np.isposinf(ref[:, 103]).all() and np.isfinite(ref).any()
    assert np.array_equal(np.isnan(score), np.isnan(ref))
    fin = np.isfinite(ref)
    assert np.array_equal(score[~fin & ~np.isnan(ref)], ref[~fin & ~np.isnan(ref)])
    assert np.allclose(score[fin], ref[fin], rtol=1e-4, atol=1e-4)
    assert np.array_equal(sel, sel_ref)


# Every row active: (sample, group) problems that divide by the XCDs (dealt round-robin when masked) and that do not, blocks of
# 32 rows without any, V packed head by head, token by token and on an odd element, no statistics without a mask
@pytest.mark.parametrize("dtype,B,nH,nG,L,dh,mask", [
    ("bf16", 8, 4, 2, 333, 64, True), ("bf16", 3, 3, 1, 385, 32, True), ("bf16", 2, 2, 2, 257, 64, False), ("f16", 4, 4, 4, 290, 32, True),
    ("bf16", 2, 4, 2, 300, 128, True), ("bf16", 1, 2, 1, 33, 64, False),
])
def test_every_row_active(dtype, B, nH, nG, L, dh, mask):
    _say(f"every row {dtype} B={B} nH={nH} L={L} dh={dh} mask={mask}")
    with sf.use_half("f16" if dtype == "f16" else "bf16"):
        for kw in (dict(), dict(strided=True), dict(v_transposed=True), dict(forced=True)):
            _gqa_case(dtype, B, nH, nG, L, dh, L, mask, seed=L, **kw)


# Masked rows of a call whose every allowed row is active: their context vector is summed from what the transposition of V leaves per
# 64 keys; a tile short of and past full, one key, several groups in a row of V, the widest head
@pytest.mark.parametrize("dtype,B,nH,nG,L,dh", [("bf16", 3, 2, 1, 63, 64), ("f16", 5, 3, 3, 64, 32), ("bf16", 5, 6, 3, 65, 32), ("bf16", 2, 4, 4, 129, 64),
                                                ("f16", 2, 4, 2, 191, 128), ("bf16", 9, 8, 2, 1100, 64)])
def test_context_where_every_allowed_row_is_active(dtype, B, nH, nG, L, dh):
    _say(f"context of masked rows {dtype} B={B} nH={nH} nG={nG} L={L} dh={dh}")
    with sf.use_half(dtype):
        for kw in (dict(), dict(strided=True)):
            _gqa_case(dtype, B, nH, nG, L, dh, L, True, seed=L, **kw)


# ... which does not look at the masked rows of V
@pytest.mark.parametrize("dtype,token_major", [("bf16", False), ("f16", True)])
def test_context_leaves_masked_values_alone(dtype, token_major):
    _say(f"masked values {dtype} token-major={token_major}")
    B, nH, nG, L, dh = 3, 4, 2, 321, 64
    g = torch.Generator(device="cuda").manual_seed(6)
    with sf.use_half(dtype):
        t = torch.bfloat16 if dtype == "bf16" else torch.float16
        Q, K, V = (torch.randn((B, n, L, dh), generator=g, device="cuda").to(t) for n in (nH, nG, nG))
        if token_major:
            V = V.transpose(1, 2).contiguous().transpose(1, 2)
        kv = (torch.rand((B, L), generator=g, device="cuda") < 0.6).to(torch.uint8)
        kv[1] = 0                                                  # no key at all: rows of zeros
        desc = sf.make_desc(B, L, nH * dh, nH, nG, dh, 64, dtype=SF_DTYPE[dtype], U_override=L)
        hg = torch.arange(nH, dtype=torch.int32, device="cuda").div(nH // nG, rounding_mode="floor").to(torch.int32).reshape(1, nH)
        clean = sf.sparse_gqa_forward(desc, Q, K, V, hg, None, kv, want_sel=False)[0]
        V[(kv == 0)[:, None, :].expand(B, nG, L)] = float("nan")
        got = sf.sparse_gqa_forward(desc, Q, K, V, hg, None, kv, want_sel=False)[0]
        torch.cuda.synchronize()
    got, clean = got[kv == 0], clean[kv == 0]
    assert bool(torch.isfinite(got).all()) and torch.equal(got, clean) and not bool(got[int((kv[0] == 0).sum()):][:L].any())


def test_value_on_an_odd_element():
    B, nH, L, dh = 2, 2, 300, 64
    rng = np.random.default_rng(4)
    Q, K, V = (to_dev(W.to_bf16_values(rng.standard_normal((B, nH, L, dh)).astype(np.float32)), "bf16") for _ in range(3))
    odd = torch.empty(V.numel() + 1, dtype=V.dtype, device="cuda")[1:].view(V.shape)
    odd.copy_(V)
    assert odd.data_ptr() % 16 == 2
    hg = torch.arange(nH, dtype=torch.int32, device="cuda").reshape(1, nH)
    for U in (-1, L):
        desc = sf.make_desc(B, L, 64, nH, nH, dh, 64, dtype=sf.SF_BF16, U_override=U)
        a, b = (sf.sparse_gqa_forward(desc, Q, K, v, hg)[0] for v in (V, odd))
        torch.cuda.synchronize()
        assert torch.equal(a, b)
