"""The kernels whose tile owns whole rows (gemm_bf16_rows.hip): the FFN in one launch and the output projection with its LayerNorm, at the
edges of their tiles and chunks, against the oracle."""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest
import torch

from paper_2604_08971_amd import binding as sf
from paper_2604_08971_amd import workloads as W
from gpu_utils import DeviceModel
from helpers import make_wl
from test_gpu_parity import _encoder_parity, _ffn_case, _say
from test_gpu_tokens_packed import _packed_case

pytestmark = pytest.mark.gpu


def _gemm_launches(run):
    torch.cuda.synchronize()
    sf.profile_begin(sf.SF_KERNEL_GEMM, 64)
    run()
    torch.cuda.synchronize()
    return sf.profile_end()[0]


# Each width; one row past a tile and one short of it; hidden channels of one and a half chunks (192 of 128, 384 of 256), of one tile
# of 64, and of a chunk and a tile; the last is one round short of full and keeps two launches
@pytest.mark.parametrize("dtype,act,B,L,d,F,keep,launches", [
    ("bf16", 0, 33, 65, 128, 200, 0.7, 1), ("f16", 1, 130, 63, 256, 300, 1.0, 1), ("bf16", 1, 120, 129, 384, 328, 1.0, 1),
    ("f16", 0, 60, 385, 512, 64, 1.0, 1), ("bf16", 0, 80, 383, 512, 576, 0.55, 1), ("bf16", 0, 75, 383, 512, 576, 0.55, 2),
])
def test_ffn_in_one_launch(monkeypatch, dtype, act, B, L, d, F, keep, launches):
    _say(f"ffn of whole rows {dtype} act={act} B={B} L={L} d={d} F={F}")
    run, counts = sf.pruned_ffn_forward, []

    def counted(*a):
        out = []
        counts.append(_gemm_launches(lambda: out.append(run(*a))))
        return out[0]

    monkeypatch.setattr(sf, "pruned_ffn_forward", counted)
    with sf.use_half(dtype):
        _ffn_case(dtype, act, B, L, d, F, keep)          # three weight sets, with and without LayerNorm and residual
    assert counts == [launches] * 2


# Two layers and a final LayerNorm: LN2 written by the output projection, the next layer's LN1 and the final one by the FFN (three launches
# a layer); missing sensors, ragged tiles, no bias to spare
@pytest.mark.parametrize("dtype,B,seg,d,Hq,Hk,dh,F", [("bf16", 20, (70, 50, 90), 128, 4, 2, 32, 256), ("f16", 65, (70, 60), 256, 4, 2, 64, 384),
                                                      ("bf16", 103, (70, 50, 90), 384, 6, 2, 64, 512), ("bf16", 103, (99, 80, 61), 512, 8, 2, 64, 640)])
def test_encoder_writes_its_layernorms_along(dtype, B, seg, d, Hq, Hk, dh, F):
    _say(f"layernorm written along {dtype} B={B} d={d}")
    spec = W.small_spec(dtype=dtype, B=B, seg=seg, d=d, Hq=Hq, Hk=Hk, dh=dh, F=F, head_keep=0.5 if d < 384 else 0.67, nl=2, c=5)
    with sf.use_half(dtype):
        wl = make_wl(spec)
        dm = DeviceModel(wl).build_plan()
        dm.forward()
        assert _gemm_launches(lambda: dm.forward()) == 6
        _encoder_parity(wl, samples=[0, B // 2, B - 1])


def _launches(kernel_class, run):
    torch.cuda.synchronize()
    sf.profile_begin(kernel_class, 64)
    run()
    torch.cuda.synchronize()
    return sf.profile_end()[0]


# Few tiles take few hidden channels (up to 5 tiles + 96 of d 128, 2048 from 192 tiles on, 32 (tiles - 116) of d 256), of which GELU makes
# a third more and empty rows of a tile as many more as they are; tiles of which more than two thirds (d 128, 256) or a half are empty take none
@pytest.mark.parametrize("dtype,act,B,L,d,F,keep,launches", [
    ("bf16", 0, 33, 64, 128, 256, 1.0, 1), ("f16", 0, 33, 64, 128, 320, 1.0, 2), ("bf16", 1, 32, 33, 128, 2048, 1.0, 2), ("f16", 1, 48, 64, 128, 192, 1.0, 1),
    ("bf16", 1, 48, 64, 128, 256, 1.0, 2), ("f16", 0, 192, 60, 128, 1920, 1.0, 1), ("f16", 0, 192, 60, 128, 1984, 1.0, 2),
    ("bf16", 0, 130, 62, 256, 384, 1.0, 1), ("bf16", 0, 130, 62, 256, 448, 1.0, 2), ("f16", 1, 290, 30, 256, 448, 1.0, 1), ("f16", 1, 290, 30, 256, 512, 1.0, 2),
    ("bf16", 0, 350, 22, 256, 64, 1.0, 1), ("bf16", 0, 350, 21, 256, 64, 1.0, 2), ("bf16", 0, 250, 65, 384, 640, 1.0, 1), ("bf16", 0, 250, 65, 384, 832, 1.0, 2),
    ("f16", 1, 250, 63, 512, 64, 1.0, 2),
])
def test_ffn_of_few_tiles(monkeypatch, dtype, act, B, L, d, F, keep, launches):
    test_ffn_in_one_launch(monkeypatch, dtype, act, B, L, d, F, keep, launches)


# ... and no LayerNorm of a launch of its own but the input's
@pytest.mark.parametrize("dtype,B,seg,d,Hq,Hk,dh,F", [("bf16", 20, (70, 50, 90), 128, 4, 2, 32, 256), ("f16", 65, (70, 60), 256, 4, 2, 64, 384),
                                                      ("bf16", 103, (70, 50, 90), 384, 6, 2, 64, 512), ("bf16", 103, (99, 80, 61), 512, 8, 2, 64, 640)])
def test_encoder_has_one_layernorm_launch(dtype, B, seg, d, Hq, Hk, dh, F):
    _say(f"one layernorm launch {dtype} B={B} L={sum(seg)} d={d}")
    spec = W.small_spec(dtype=dtype, B=B, seg=seg, d=d, Hq=Hq, Hk=Hk, dh=dh, F=F, head_keep=0.5 if d < 384 else 0.67, nl=2, c=5)
    with sf.use_half(dtype):
        dm = DeviceModel(make_wl(spec)).build_plan()
        assert _launches(sf.SF_KERNEL_LAYERNORM, dm.forward) == 1


def _first_samples(wl, n):
    return dataclasses.replace(wl, x=wl.x[:n], presence=wl.presence[:n], pattern_id=wl.pattern_id[:n])


# A sample's output does not depend on how many others there are, to the bit: few of them go through separate launches, all of them
# through the whole-row kernels, whose products and row sums run in the same order.  Two layers, so that LN2, the next layer's LN1 and the
# final LayerNorm are all written along.  Sizes at which both sides' separate launches would slice K alike and no LayerNorm
# rides along with the product that reads it (in the last case all do, as they do among few): one chain (d 384, 512; the second without
# biases); projection and FFN in slices, of up to three tiles, up-projection of one chain and sliced; four slices of an odd number of
# tiles; four in the projection alone; short samples of d 384, which are sliced, for which the wide tiles have no registers.
@pytest.mark.parametrize("dtype,few,B,L,d,Hq,Hk,dh,F,act,keep,launches", [
    ("bf16", 60, 80, 383, 384, 6, 2, 64, 512, 0, 0.75, (8, 6)), ("f16", 60, 80, 383, 512, 8, 2, 64, 320, 1, 0.75, (8, 6)),
    ("bf16", 78, 79, 62, 128, 8, 1, 32, 640, 0, 0.75, (8, 6)), ("f16", 41, 42, 62, 128, 8, 1, 32, 320, 1, 0.75, (8, 6)),
    ("bf16", 134, 135, 62, 256, 8, 1, 32, 448, 1, 0.25, (8, 6)), ("f16", 127, 128, 50, 256, 8, 1, 32, 256, 0, 0.25, (8, 6)),
    ("bf16", 127, 128, 50, 256, 8, 1, 32, 192, 1, 0.25, (8, 6)), ("bf16", 63, 64, 50, 256, 8, 1, 32, 192, 0, 0.75, (8, 8)),
    ("bf16", 31, 32, 50, 128, 8, 1, 32, 64, 0, 0.25, (8, 8)), ("f16", 180, 220, 35, 384, 6, 2, 64, 2048, 0, 0.75, (8, 8)),
])
def test_same_bits_as_separate_launches(dtype, few, B, L, d, Hq, Hk, dh, F, act, keep, launches):
    _say(f"bits of whole rows {dtype} few={few} B={B} L={L} d={d} F={F}")
    spec = W.small_spec(dtype=dtype, B=B, seg=(L // 2, L - L // 2), extra=0, d=d, Hq=Hq, Hk=Hk, dh=dh, F=F, head_keep=keep, ffn_keep=1.0, nl=2,
                        act=act, final_ln=True)
    with sf.use_half(dtype):
        wl = W.make_workload(spec)
        # rows far from zero, whose last bits the order of a sum decides
        wl = dataclasses.replace(wl, x=W.storage_rounding(dtype)(wl.x + np.random.default_rng(L).normal(0, 30, (B, L, 1))))
        got, seen = [], []
        for n in (few, B):
            dm = DeviceModel(_first_samples(wl, n))
            if d == 512:
                dm.dense = [{k: v for k, v in w.items() if k not in ("bq", "bk", "bv", "bo", "b1", "b2")} for w in dm.dense]
            dm.build_plan()
            dm.forward()
            seen.append(_gemm_launches(lambda: got.append(dm.forward()[0][:few].clone())))
        assert tuple(seen) == launches
        assert bool(torch.isfinite(got[0]).all())
        assert int((got[0] != got[1]).sum()) == 0


# One weight set and no pattern numbers: the samples are one long one, and tiles cross their ends.  The same bits as sample by sample (products
# of one chain on both sides), a last tile of 44 and of 53 rows; and a NaN, an infinity and a value whose square overflows stay
# in their own sample.
@pytest.mark.parametrize("dtype,B,L,d,Hq,Hk,dh,F", [("bf16", 100, 131, 256, 4, 2, 64, 320), ("f16", 83, 383, 512, 8, 2, 64, 320)])
def test_samples_joined(dtype, B, L, d, Hq, Hk, dh, F):
    _say(f"whole rows of joined samples {dtype} B={B} L={L} d={d}")
    spec = W.small_spec(dtype=dtype, B=B, seg=(L - 60, 60), extra=0, d=d, Hq=Hq, Hk=Hk, dh=dh, F=F, head_keep=0.5, ffn_keep=1.0, nl=2, dropout="none")
    with sf.use_half(dtype):
        dm = DeviceModel(W.make_workload(spec)).build_plan()
        one_by_one = dm.forward()[0].clone()
        dm.pattern_id = None
        assert _gemm_launches(dm.forward) == 6 and _launches(sf.SF_KERNEL_LAYERNORM, dm.forward) == 1
        joined = dm.forward()[0].clone()
        assert bool(torch.isfinite(joined).all()) and int((joined != one_by_one).sum()) == 0
        bad = {B // 3: float("nan"), B // 2: float("inf"), B - 1: 6e4 if dtype == "f16" else 2e38}
        for b, v in bad.items():
            dm.x[b, 7, 3] = v
        Y = dm.forward()[0]
        others = [b for b in range(B) if b not in bad]
        assert int((Y[others] != joined[others]).sum()) == 0


# Packed rows, whose blocks of 256 may be unused or straddle samples: the widths with one workgroup per compute unit
@pytest.mark.parametrize("dtype,B,d,Hq", [("bf16", 165, 384, 6), ("bf16", 165, 512, 8)])
def test_packed_rows(monkeypatch, dtype, B, d, Hq):
    _say(f"whole rows packed {dtype} B={B} d={d}")
    run, counts = sf.encoder_forward_packed, []

    def counted(*a, **kw):
        counts.extend(_launches(c, lambda: run(*a, **kw)) for c in (sf.SF_KERNEL_GEMM, sf.SF_KERNEL_LAYERNORM))
        return run(*a, **kw)

    monkeypatch.setattr(sf, "encoder_forward_packed", counted)
    _packed_case(make_wl(W.small_spec(dtype=dtype, d=d, Hq=Hq, Hk=2, dh=64, F=320, seg=(130, 70, 60), B=B, nl=2, dropout="upto:2", c=5)),
                 samples=[0, B // 2, B - 1])
    assert counts == [6, 1]


# What the whole-row kernels refuse: an output, or the vectors of LN2 or the final LayerNorm, off their 16 bytes.  The launches take over; rows
# beside the output stay as they are.
@pytest.mark.parametrize("dtype,B,L,d,dh", [("bf16", 12, 300, 128, 32), ("f16", 80, 383, 512, 64)])
@pytest.mark.parametrize("what,layernorms", [("Y", 2), ("ln2_g", 2), ("ln2_b", 2), ("final", 2)])
def test_off_alignment(dtype, B, L, d, dh, what, layernorms):
    _say(f"whole rows off alignment {what} {dtype} B={B} L={L} d={d}")
    spec = W.small_spec(dtype=dtype, B=B, seg=(L - 60, 60), extra=0, d=d, Hq=d // dh, Hk=1, dh=dh, F=320, head_keep=0.5, ffn_keep=1.0, nl=1, dropout="none")

    def moved(t, by):
        buf = torch.full((t.numel() + 16,), 7.0, dtype=t.dtype, device="cuda")
        v = buf[by:by + t.numel()].view(t.shape)
        v.copy_(t)
        return buf, v

    with sf.use_half(dtype):
        dm = DeviceModel(W.make_workload(spec)).build_plan()
        assert _launches(sf.SF_KERNEL_LAYERNORM, dm.forward) == 1
        ref = dm.forward()[0]
        for by in (1, 4):                                          # 2 and 8 bytes
            out, hold = None, []
            if what == "Y":
                buf, out = moved(ref, by)
            else:
                dm = DeviceModel(W.make_workload(spec))
                vectors = dm.final_ln if what == "final" else dm.dense[0]
                for n in (("g", "b") if what == "final" else (what,)):
                    b, vectors[n] = moved(vectors[n], by)
                    hold.append(b)
                dm.build_plan()
            assert _launches(sf.SF_KERNEL_LAYERNORM, lambda: dm.forward(out=out)) == layernorms
            got = dm.forward(out=out)[0]
            # the LayerNorm of rows off their alignment adds in another order: one code in some thousand moves by a place, and what a moved
            # LN2 code moves in the FFN is less than that of the sum
            place = 2.0 ** (-7 if dtype == "bf16" else -10)
            diff = (got.float() - ref.float()).abs()
            assert float((diff / ref.float().abs().clamp(min=1)).max()) <= 2 * place and float((diff != 0).float().mean()) < 0.01
            if what == "Y":
                assert bool((buf[:by] == 7).all()) and bool((buf[by + ref.numel():] == 7).all())
