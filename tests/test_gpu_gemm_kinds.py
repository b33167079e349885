"""The bf16 GEMM kernels that take what the 256 x 256 tiles do not: K slices (a few tiles) and 128 x 128 tiles, at the
edges of their tiles and at a K tail of half a K tile, through the pruned FFN and the encoder against the oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2604_08971_amd import binding as sf
from paper_2604_08971_amd import workloads as W
from gpu_utils import SF_DTYPE, DeviceModel, desc_for, layernorm_as_launched, to_dev, to_host
from helpers import err_metric, make_wl
from test_gpu_parity import _encoder_parity, _ffn_case, _moe_case, _say

pytestmark = pytest.mark.gpu


# 32 x 64 and 64 x 64 slices: one row, one row past a tile, K of one tile / one and a half (d = 96) / more tiles than
# slices; 128 x 128 tiles: one row short of and past a tile, widths that are no multiple of it, K tails
@pytest.mark.parametrize("act,B,L,d,F,keep", [
    (0, 1, 1, 64, 64, 1.0), (1, 1, 33, 96, 200, 0.5), (0, 2, 129, 96, 200, 0.7), (0, 1, 65, 640, 1280, 0.6),
    (1, 4, 512, 512, 1024, 0.6), (0, 30, 127, 320, 1000, 0.64), (1, 30, 129, 352, 1000, 0.64), (0, 300, 1, 64, 136, 1.0),
])
def test_ffn_on_small_tiles(act, B, L, d, F, keep):
    _say(f"small tiles act={act} B={B} L={L} d={d} F={F}")
    _ffn_case("bf16", act, B, L, d, F, keep)


# Which kernel takes a problem is an estimate: the choice is asserted, so that the remainders of each kernel stay covered
# (up-projection, down-projection; K tails in the up-projections)
@pytest.mark.parametrize("act,B,L,d,F,keep,up,down", [
    (0, 4, 129, 352, 1000, 1.0, "slices4", "slices8"), (1, 2, 513, 480, 640, 1.0, "slices4", "slices4"),
    (1, 1, 33, 96, 200, 0.5, "slices8", "slices8"), (0, 30, 129, 352, 1000, 0.64, "128x128", "128x128"),
    (0, 1, 193, 72, 72, 1.0, "generic", "slices8"), (0, 16, 2100, 512, 2048, 0.6, "256x256", "128x128"),
])
def test_ffn_on_each_kernel(act, B, L, d, F, keep, up, down):
    _say(f"gemm kernels act={act} B={B} L={L} d={d} F={F}: {up}, {down}")
    desc = sf.make_desc(B, L, d, 8, 2, 8, F, P=3, dtype=sf.SF_BF16)
    Fp = sf.ffn_padded(desc, max(1, int(keep * F + 0.5)))
    assert (sf.gemm_kernel(desc, Fp, d, act + 1), sf.gemm_kernel(desc, d, Fp)) == (up, down)
    if B * L < 8000:                             # the largest case is covered at its size elsewhere
        _ffn_case("bf16", act, B, L, d, F, keep)


# K = kept heads x 32: an odd number of heads leaves a K tail in the output projection; ragged lengths in the transposed
# column range of the Q/K/V projection, with slices (B = 2) and 128 x 128 tiles (B = 40)
@pytest.mark.parametrize("dtype,B,seg,drop", [("bf16", 2, (70, 50, 91), "bernoulli:0.3"), ("bf16", 40, (170, 91), "none"),
                                              ("f16", 3, (33, 95), "none")])
def test_encoder_with_an_odd_number_of_heads(dtype, B, seg, drop):
    _say(f"odd heads {dtype} B={B} seg={seg}")
    spec = W.small_spec(dtype=dtype, B=B, seg=seg, d=128, Hq=4, Hk=2, dh=32, F=256, head_keep=0.75, nl=2, dropout=drop)
    with sf.use_half("f16" if dtype == "f16" else "bf16"):
        _encoder_parity(make_wl(spec))


# MoE block: token rows read through a map, expert widths that end a tile early (n_lim, k_lim), K tails of half a K tile
# (d % 64 == 32), with and without the LayerNorm that would otherwise hand over a padded copy of X
@pytest.mark.parametrize("dtype,B,seg,d,F,E,k,up", [("bf16", 3, (70, 50, 9), 96, 200, 4, 2, "128x128"), ("f16", 2, (33, 95), 96, 136, 5, 1, "slices8"),
                                                    ("bf16", 9, (700, 333), 160, 640, 8, 2, "128x128"), ("f16", 9, (700, 333), 160, 640, 4, 3, "128x128")])
def test_moe_on_small_tiles(dtype, B, seg, d, F, E, k, up):
    _say(f"moe on small tiles {dtype} B={B} d={d} F={F} E={E}")
    wl = make_wl(W.small_spec(dtype=dtype, B=B, seg=seg, d=d, dh=32, F=F, dropout="upto:1"))
    # 256-row blocks of one (pattern, expert) each
    blocks = (wl.x.shape[0] * wl.spec.L * k + 255) // 256 + wl.P * E
    desc = sf.make_desc(blocks, 256, d, 8, 2, 8, F, P=2, dtype=sf.SF_F16 if dtype == "f16" else sf.SF_BF16)
    with sf.use_half("f16" if dtype == "f16" else "bf16"):
        assert sf.gemm_kernel(desc, sf.ffn_padded(desc, int(W.make_moe_block(wl, E, k).k_ffn.max())), d, 1) == up
        _moe_case(wl, E, k, pre_ln=False)
        _moe_case(wl, E, k, forced=True)


# a caller's X that starts on an odd element, which the loads straight into LDS do not take: few rows and many
@pytest.mark.parametrize("B,L,d,F", [(1, 33, 96, 200), (2, 300, 256, 512)])
def test_ffn_on_a_misaligned_input(B, L, d, F):
    _say(f"misaligned X B={B} L={L} d={d} F={F}")
    wl = make_wl(W.small_spec(dtype="bf16", B=B, seg=(L - 1,), extra=1, d=d, Hq=2, Hk=1, dh=32, F=F, nl=1, dropout="none", final_ln=False))
    dm = DeviceModel(wl).build_plan()
    X = dm.x.view(B * L, d)
    odd = torch.empty(X.numel() + 8, dtype=X.dtype, device="cuda")[1:X.numel() + 1].view(B * L, d)
    odd.copy_(X)
    assert odd.data_ptr() % 16 == 2
    for res in (True, False):
        ref, got = (sf.pruned_ffn_forward(dm.desc, dm.layers[0], x, dm.pattern_id, False, res) for x in (X, odd))
        torch.cuda.synchronize()
        # the same rounding points, sums in another order: one unit of the hidden activations and of the output
        assert err_metric(to_host(got), to_host(ref)) <= 2.0 ** -6


# The LayerNorm that rides along with few rows: one row, one past a tile, one and two K tiles per slice (d 64 .. 1024), the last
# number of tiles that takes it and the first that does not (16 x 16 and 17 x 16 tiles); rows far from zero, whose
# variance a sum of squares would lose.  Against the FFN of rows normalised in 64 bits: both round them to 16 bits, a last
# place apart at most where the exact value lies between two numbers, so the outputs differ by less than one rounding of the
# hidden activations and of the output.
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B,L,d,F", [(1, 1, 64, 64), (1, 33, 64, 200), (3, 65, 512, 520), (1, 31, 576, 640), (2, 40, 1024, 1000),
                                     (1, 512, 256, 1024), (1, 513, 256, 1024)])
def test_ffn_with_layernorm_along(dtype, B, L, d, F):
    _say(f"layernorm along {dtype} B={B} L={L} d={d} F={F}")
    with sf.use_half(dtype):
        wl = make_wl(W.small_spec(dtype=dtype, B=B, seg=(max(1, L - 1),), extra=int(L > 1), d=d, Hq=2, Hk=1, dh=32, F=F, nl=1, ffn_keep=1.0,
                                  dropout="none", final_ln=False))
        dm = DeviceModel(wl).build_plan()
        lay = dm.layers[0]
        g = torch.Generator(device="cuda").manual_seed(L)
        x = torch.randn((B * L, d), generator=g, device="cuda") + torch.randn((B * L, 1), generator=g, device="cuda") * 50
        x = x.to(dm.x.dtype)
        gamma, beta = (lay.dense[n].double() for n in ("ln2_g", "ln2_b"))
        xn = torch.nn.functional.layer_norm(x.double(), (d,), gamma, beta, 1e-5).to(x.dtype)
        got = sf.pruned_ffn_forward(dm.desc, lay, x, dm.pattern_id, True, False)
        ref = sf.pruned_ffn_forward(dm.desc, lay, xn, dm.pattern_id, False, False)
        torch.cuda.synchronize()
        assert err_metric(to_host(got), to_host(ref)) <= (2.0 ** -6 if dtype == "bf16" else 2.0 ** -9)


# The same in fp32 (rows of at most 256, at most 1024 tiles of 32 x 32): one row, one past a tile, one and several K steps, a last step
# that is not full; the longest row that takes it, the first that does not, and a launch with too many tiles.  Rows far from zero:
# their mean of 50 is exact to 50 * 2^-24, and so is every normalised value to about that; eight of those bound what the two
# products, whose weights have unit norm, make of it next to their own rounding.
@pytest.mark.parametrize("B,L,d,F", [(1, 1, 8, 16), (2, 33, 64, 128), (1, 65, 200, 72), (3, 31, 256, 64), (2, 40, 264, 64), (40, 130, 64, 200)])
def test_f32_ffn_with_layernorm_along(B, L, d, F):
    _say(f"layernorm along f32 B={B} L={L} d={d} F={F}")
    wl = make_wl(W.small_spec(dtype="f32", B=B, seg=(max(1, L - 1),), extra=int(L > 1), d=d, Hq=2, Hk=1, dh=8, F=F, nl=1, ffn_keep=1.0,
                              dropout="none", final_ln=False))
    dm = DeviceModel(wl).build_plan()
    lay = dm.layers[0]
    g = torch.Generator(device="cuda").manual_seed(L)
    x = torch.randn((B * L, d), generator=g, device="cuda") + torch.randn((B * L, 1), generator=g, device="cuda").sign() * 50
    got = sf.pruned_ffn_forward(dm.desc, lay, x, dm.pattern_id, True, False)
    w = {n: lay.dense[n].double() for n in ("ln2_g", "ln2_b", "W1", "b1", "W2", "b2")}
    xn = torch.nn.functional.layer_norm(x.double(), (d,), w["ln2_g"], w["ln2_b"], 1e-5)
    ref = torch.relu(xn @ w["W1"].T + w["b1"]) @ w["W2"] + w["b2"]
    torch.cuda.synchronize()
    assert err_metric(to_host(got), ref.cpu().numpy()) <= 8 * 50 * 2.0 ** -24


# ... with the bits of the launch: few rows take it along, many (more than 1024 tiles) do not.  Chunks of eight columns of which a lane has
# one, some lanes none, all four; rows that are no whole chunks, and longer than one, two and three columns per lane
@pytest.mark.parametrize("d", [24, 64, 200, 256, 36, 250, 190, 100])
def test_f32_layernorm_along_has_the_bits_of_the_launch(d):
    _say(f"layernorm along f32 bits d={d}")
    few, B, L, F = 2, 36, 130, 192
    wl = make_wl(W.small_spec(dtype="f32", B=B, seg=(L,), extra=0, d=d, Hq=2, Hk=1, dh=8, F=F, nl=1, ffn_keep=1.0, dropout="none", final_ln=False))
    dm = DeviceModel(wl).build_plan()
    g = torch.Generator(device="cuda").manual_seed(d)
    x = torch.randn((B * L, d), generator=g, device="cuda") + 50 * torch.randn((B * L, 1), generator=g, device="cuda")
    got = [sf.pruned_ffn_forward(desc_for(wl, B=n), dm.layers[0], x[:n * L], dm.pattern_id[:n], True, False)[:few * L] for n in (few, B)]
    assert int((got[0] != got[1]).sum()) == 0


# Behind the last column nothing is added up: a constant row is its mean (2^122: every sum of 24 or 36 is exact), whose multiple by 1 / sqrt(eps)
# would overflow there, and its output is what the bias of the LayerNorm gives
@pytest.mark.parametrize("d", [24, 36])
def test_f32_layernorm_along_of_a_constant_row(d):
    _say(f"layernorm along f32 constant row d={d}")
    wl = make_wl(W.small_spec(dtype="f32", B=1, seg=(3,), extra=0, d=d, Hq=2, Hk=1, dh=8, F=64, nl=1, ffn_keep=1.0, dropout="none", final_ln=False))
    dm = DeviceModel(wl).build_plan()
    x = torch.zeros((3, d), device="cuda")
    x[1] = 2.0 ** 122
    got = sf.pruned_ffn_forward(dm.desc, dm.layers[0], x, dm.pattern_id, True, False)
    assert bool(torch.isfinite(got).all()) and torch.equal(got[1], got[0])


# The router that takes the LayerNorm along: rows of one and two chunks of 512 and just beyond (a launch of its own), up to 8 and 16 experts
# and beyond, blocks of 16 tokens (one short of full, full, one more) and of 64
@pytest.mark.parametrize("dtype,B,L,d,E,k", [("bf16", 1, 15, 512, 8, 2), ("f16", 1, 16, 520, 9, 2), ("bf16", 1, 17, 1024, 16, 3), ("f16", 3, 33, 1032, 4, 1),
                                             ("bf16", 2, 50, 64, 17, 2), ("bf16", 129, 128, 64, 8, 2)])
def test_moe_router_with_layernorm_along(dtype, B, L, d, E, k):
    _say(f"moe router {dtype} B={B} L={L} d={d} E={E}")
    wl = make_wl(W.small_spec(dtype=dtype, B=B, seg=(L - 5, 3), extra=2, d=d, Hq=2, Hk=1, dh=32, F=128, dropout="upto:1"))
    with sf.use_half(dtype):
        _moe_case(wl, E, k)


# Few tokens and many (pattern, expert) pairs: most of the router's blocks only clear what the sort starts from
@pytest.mark.parametrize("B,seg,P,E", [(3, (1,) * 6, 64, 16), (40, (2, 1, 1, 2, 1, 2), 40, 5)])
def test_moe_of_few_tokens_and_many_pairs(B, seg, P, E):
    _say(f"moe of few tokens B={B} P={P} E={E}")
    wl = make_wl(W.small_spec(dtype="bf16", B=B, seg=seg, extra=0, d=64, Hq=2, Hk=1, dh=32, F=64, dropout="none"))
    wl.pattern_bits = np.arange(P)
    wl.pattern_id = np.random.default_rng(P).integers(0, P, B).astype(np.int32)
    _moe_case(wl, E, 2)


# A LayerNorm that rides along with the router gives the bits of the launch it replaces (17 experts: that launch): the block without one on
# rows normalised like it.  Means of 30, so that a row's sums decide its last bits.
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d,E", [(384, 4), (768, 16), (384, 17)])
def test_moe_layernorm_along_has_the_bits_of_the_launch(dtype, d, E):
    _say(f"moe layernorm bits {dtype} d={d} E={E}")
    B, L, F, k = 3, 700, 64, 2
    wl = make_wl(W.small_spec(dtype=dtype, B=B, seg=(L - 5, 3), extra=2, d=d, Hq=2, Hk=1, dh=32, F=F, dropout="none"))
    mb = W.make_moe_block(wl, E, k)
    rnd = W.storage_rounding(dtype)
    X = rnd(wl.x.reshape(B * L, d) + np.random.default_rng(d).normal(0, 30, (B * L, 1)))
    with sf.use_half(dtype):
        dt = SF_DTYPE[dtype]
        masks = sf.gate_scores_to_masks(sf.make_desc(B, L, d, 8, 2, 8, F, n_layers=E, P=1, dtype=dt), to_dev(np.zeros((E, 1, 8), np.float32), "f32"),
                                        to_dev(mb.g_ffn, "f32"), [1] * E, mb.k_ffn.tolist())
        desc = sf.make_desc(B, L, d, 8, 2, 8, F, n_layers=1, P=1, dtype=dt)
        cm = sf.compact_moe_experts(desc, {n: to_dev(v, dtype) for n, v in mb.dense.items()}, masks["ffn_idx"], k, mb.k_ffn.tolist())
        got = sf.moe_ffn_forward(desc, cm, to_dev(X, dtype), None, pre_ln=True, add_residual=False, want_route=True)
        xn = layernorm_as_launched(X, mb.dense["ln_g"], mb.dense["ln_b"], dtype)
        ref = sf.moe_ffn_forward(desc, cm, to_dev(xn, dtype), None, pre_ln=False, add_residual=False, want_route=True)
        torch.cuda.synchronize()
    assert [int((a != b).sum()) for a, b in zip(got, ref)] == [0, 0, 0, 0]
