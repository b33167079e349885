"""Performance cases of the pruned multimodal encoder: what a program that uses this package has it do, through the
public entry points of `paper_2604_08971_amd.binding`, on synthetic inputs made on the GPU.

A case is a dict of plain values.  `kind` says which calls a pass makes:

  encoder   allowed keys from the presence masks, then the encoder forward (with `plan`: masks and compacted weights are
            rebuilt first, as when the platform's keep set changes from batch to batch)
  fp8       the encoder with FFNs and attention projections in FP8 arithmetic
  packed    pack the present tokens of all samples, encoder over the packed rows, unpack
  gqa       sparse grouped-query attention alone
  moe       the Sparse-MoE FFN block with pruned experts
  gate      the keep sets of a new platform budget: gate scores, budget search, keep masks

`seg` lists the tokens of each modality ("256+128+64+32"), `fusion` the always-present tokens behind them; at most
`max_drop` modalities are missing in a sample and every such presence pattern has its own compacted weights.
"""
import itertools
import math

import torch

from paper_2604_08971_amd import binding as sf

_TORCH = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
_SF = {"bf16": sf.SF_BF16, "f16": sf.SF_F16, "f32": sf.SF_F32}


def _encoder(name, kind="encoder", dtype="bf16", B=1, seg="512", fusion=0, max_drop=0, d=512, Hq=8, Hk=2, dh=64, F=2048,
             nl=1, head_keep=0.7, ffn_keep=0.6, c=5, act="relu", final_ln=False, n_sample=0, plan=False):
    case = dict(kind=kind, dtype=dtype, B=B, seg=seg, fusion=fusion, max_drop=max_drop, d=d, Hq=Hq, Hk=Hk, dh=dh, F=F,
                nl=nl, head_keep=head_keep, ffn_keep=ffn_keep, c=c, act=act, final_ln=final_ln, n_sample=n_sample, plan=plan)
    return dict(case, name=name) if name else case


def listed():
    return [
        # The smallest model of the repository (C1): a wearable classifier in fp32, two windows of three sensors.
        # Launches and latency are all there is.
        _encoder("tiny_f32", dtype="f32", B=2, seg="16+16+16", max_drop=1, d=64, Hq=4, Hk=2, dh=16, F=256, head_keep=0.5,
                 ffn_keep=0.5),
        # Online inference: one window at a time through the six-layer stack (C4's model), where the answer is waited for.
        _encoder("one_window", B=1, seg="170+170+170", fusion=2, nl=6, head_keep=0.75, final_ln=True),
        # A small batch with sensor dropout (C2), plan and forward: what a step costs when the keep sets change.
        _encoder("small_step", B=64, seg="128+128+128", max_drop=2, d=256, Hq=8, Hk=2, dh=32, F=1024, head_keep=0.75,
                 plan=True),
        # Four sensors at different rates, up to two of them missing (C3), the plan kept.
        _encoder("dropout_batch", B=256, seg="256+128+64+32", max_drop=2, Hk=4, head_keep=0.5, ffn_keep=0.5),
        # The deepest stack at a full batch (C4): the most work of all.
        _encoder("stack", B=128, seg="170+170+170", fusion=2, nl=6, head_keep=0.75, final_ln=True),
        # The headline workload (C5): long sequences, plan and forward in one step.
        _encoder("long_step", B=16, seg="2048+2048", d=768, Hq=12, Hk=4, F=3072, ffn_keep=0.7, plan=True),
        # The same layer as an FP8 model.
        _encoder("long_fp8", kind="fp8", B=16, seg="2048+2048", d=768, Hq=12, Hk=4, F=3072, ffn_keep=0.7),
        # The dropout batch with the tokens of missing sensors left out instead of masked.
        _encoder("packed_batch", kind="packed", B=256, seg="256+128+64+32", max_drop=2, Hk=4, head_keep=0.5, ffn_keep=0.5),
        # An FP16 model on odd lengths: GELU, the sampled sparsity score, two layers and a final LayerNorm.
        _encoder("ragged_f16", dtype="f16", B=37, seg="577+301+143", max_drop=1, d=384, Hq=12, Hk=4, dh=32, F=1536, nl=2,
                 act="gelu", final_ln=True, n_sample=64),
        # Attention alone, every query active (the dense comparison), an odd length and a missing sensor.
        dict(name="dense_attention", kind="gqa", dtype="bf16", B=8, seg="1000+777", fusion=0, max_drop=1, nH=8, nG=4,
             dh=64, c=5, dense=True),
        # The Sparse-MoE block: eight experts, two per token, on the tokens of the long workload.
        dict(name="moe_block", kind="moe", dtype="bf16", B=16, seg="2048+2048", fusion=0, max_drop=0, d=768, F=3072,
             experts=8, top_k=2, act="relu"),
        # A new platform budget for the six-layer stack with every presence pattern of three sensors: scores, threshold and
        # masks; the host reads the counts in between, since the buffers of the compacted weights are sized with them.
        dict(name="gate_plan", kind="gate", dtype="bf16", B=1, seg="170+170+170", fusion=2, max_drop=2, d=512, Hq=8, Hk=2,
             dh=64, F=2048, nl=6, hidden=16, budget=0.6, c=5),
    ]


# ------------------------------------------------------------------------------------------------ sizes of a case
def _patterns(n_mod, max_drop):
    """Presence bit patterns with at most max_drop modalities missing, ascending."""
    every = (1 << n_mod) - 1
    miss = [m for k in range(max_drop + 1) for m in itertools.combinations(range(n_mod), k)]
    return sorted(every & ~sum(1 << j for j in m) for m in miss)


def _segments(case):
    return [int(t) for t in case["seg"].split("+")]


def _length(case):
    return sum(_segments(case)) + case["fusion"]


def _keep(ratio, n):
    return max(1, min(n, int(math.floor(ratio * n + 0.5))))


def _active(L, c):
    return min(L, c * math.ceil(math.log(L)))


def _mean_allowed(case):
    """Expected number, and expected square, of the allowed keys of a sample: the number of missing modalities is uniform in
    0..max_drop, then which ones they are."""
    seg, n1, n2 = _segments(case), 0.0, 0.0
    for k in range(case["max_drop"] + 1):
        combos = list(itertools.combinations(seg, k))
        for miss in combos:
            n = _length(case) - sum(miss)
            n1 += n / len(combos) / (case["max_drop"] + 1)
            n2 += n * n / len(combos) / (case["max_drop"] + 1)
    return n1, n2


# ------------------------------------------------------------------------------------------------ drawn cases
def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _split(rng, L, n_mod):
    """L tokens over n_mod sensors at rates that differ by up to four."""
    w = [math.exp(rng.uniform(0.0, math.log(4.0))) for _ in range(n_mod)]
    seg = [max(1, int(L * x / sum(w))) for x in w]
    seg[0] += max(0, L - sum(seg))
    return "+".join(str(s) for s in seg)


def _draw_encoder(rng, kind):
    dtype = "bf16" if kind in ("fp8", "packed") else rng.choice(["bf16", "bf16", "bf16", "f16", "f32"])
    n_mod = rng.randint(2, 4)
    if dtype == "f32":                        # small models only: the fp32 path is there for them
        Hq = rng.choice([2, 4, 8])
        dh = rng.choice([8, 16, 32])
        L, B, nl = _log_int(rng, 24, 256), _log_int(rng, 1, 16), rng.randint(1, 2)
    else:
        Hq = rng.choice([8, 12, 16] if kind == "fp8" else [4, 6, 8, 12, 16])
        dh = rng.choice([32, 64])
        L = _log_int(rng, 256 if kind == "fp8" else 96 if kind == "packed" else 48, 4096)
        B = _log_int(rng, 1, 256)
        nl = 1 if kind == "fp8" else rng.choice([1, 1, 2, 4, 6])   # FP8: one calibrated layer, as in the benchmark
    d = min(1024, Hq * dh)
    Hk = rng.choice([g for g in (1, 2, 4) if Hq % g == 0])
    if kind == "fp8":
        d = max(256, d // 128 * 128)
    case = _encoder(None, kind=kind, dtype=dtype, B=B, seg=_split(rng, L, n_mod), fusion=rng.choice([0, 0, 1, 2]),
                    max_drop=rng.randint(1, min(2, n_mod - 1)) if kind == "packed" else rng.randint(0, min(2, n_mod - 1)),
                    d=d, Hq=Hq, Hk=Hk, dh=dh, F=4 * d, nl=nl, head_keep=round(rng.uniform(0.5, 0.9), 2),
                    ffn_keep=round(rng.uniform(0.4, 0.8), 2), act=rng.choice(["relu", "relu", "gelu"]),
                    final_ln=nl > 1, n_sample=rng.choice([0, 0, 0, 64]) if kind == "encoder" and L >= 256 else 0,
                    plan=kind == "encoder" and rng.random() < 0.3)
    return case


def draw(rng):
    kind = rng.choice(["encoder"] * 6 + ["fp8", "packed", "gqa", "moe", "gate"])
    if kind in ("encoder", "fp8", "packed"):
        case = _draw_encoder(rng, kind)
        most = 2.0e9 if case["dtype"] == "f32" else 8.0e11
        while work(case)["flops"] > most or case["B"] * _length(case) > 131072:
            case["B"] = max(1, case["B"] // 2)
            if case["B"] == 1 and work(case)["flops"] > most:
                case["nl"] = 1
                case["final_ln"] = False
                break
        return case
    if kind == "gqa":
        nG = rng.choice([1, 2, 4])
        n_mod = rng.randint(1, 3)
        case = dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "f16"]), B=_log_int(rng, 1, 64),
                    seg=_split(rng, _log_int(rng, 128, 4096), n_mod), fusion=0, max_drop=rng.randint(0, min(1, n_mod - 1)),
                    nH=nG * rng.choice([1, 2, 3]), nG=nG, dh=rng.choice([32, 64, 64]), c=5, dense=rng.random() < 0.5)
        while work(case)["flops"] > 4.0e11:
            case["B"] = max(1, case["B"] // 2)
        return case
    if kind == "moe":
        d = rng.choice([256, 384, 512, 768])
        case = dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "f16"]), B=_log_int(rng, 1, 64),
                    seg=_split(rng, _log_int(rng, 64, 2048), 2), fusion=0, max_drop=rng.randint(0, 1), d=d, F=4 * d,
                    experts=rng.choice([4, 8, 16]), top_k=rng.randint(1, 2), act="relu")
        while work(case)["flops"] > 6.0e11 or case["B"] * _length(case) > 65536:
            case["B"] = max(1, case["B"] // 2)
        return case
    Hq, dh, n_mod = rng.choice([4, 8, 12]), rng.choice([32, 64]), rng.randint(2, 4)
    d = Hq * dh
    return dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "f16"]), B=1, seg=_split(rng, _log_int(rng, 64, 2048), n_mod),
                fusion=rng.choice([0, 2]), max_drop=rng.randint(0, min(2, n_mod - 1)), d=d, Hq=Hq,
                Hk=rng.choice([g for g in (2, 4) if Hq % g == 0]), dh=dh, F=4 * d, nl=rng.randint(1, 6), hidden=16,
                budget=round(rng.uniform(0.4, 0.8), 2), c=5)


# ------------------------------------------------------------------------------------------------ inputs
class _Gen:
    """Seeded tensors on the GPU with the distributions of a trained layer's tensors at initialisation scale."""

    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda").manual_seed(seed)
        self.dt = _TORCH[dtype]

    def normal(self, shape, std=1.0, base=0.0, dtype=None):
        t = torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32)
        return t.mul_(std).add_(base).to(dtype or self.dt)

    def uniform(self, shape):
        return torch.rand(shape, generator=self.g, device="cuda", dtype=torch.float32)


def _presence(case, seed):
    """Host: presence [B, M] and the pattern index of every sample (a data loader knows both)."""
    import numpy as np
    rng = np.random.Generator(np.random.PCG64([seed, 17]))
    M, pats = len(_segments(case)), _patterns(len(_segments(case)), case["max_drop"])
    pres = np.ones((case["B"], M), dtype=np.uint8)
    for b in range(case["B"]):
        k = int(rng.integers(0, case["max_drop"] + 1))
        pres[b, rng.choice(M, size=k, replace=False)] = 0
    bits = (pres.astype(np.int64) << np.arange(M)).sum(axis=1)
    return pres, np.searchsorted(np.array(pats), bits).astype(np.int32), pats


def _inputs(case, seed, st):
    """Presence masks, token map and pattern numbers on the device."""
    import numpy as np
    pres, pid, pats = _presence(case, seed)
    seg = _segments(case)
    tok = np.concatenate([np.full(n, m, dtype=np.int32) for m, n in enumerate(seg)] + [np.full(case["fusion"], -1, np.int32)])
    st["presence"], st["tok"] = torch.from_numpy(pres).cuda(), torch.from_numpy(tok).cuda()
    st["pid"] = torch.from_numpy(pid).cuda() if len(pats) > 1 else None
    st["patterns"] = torch.tensor(pats, dtype=torch.int32, device="cuda")
    return pres, pid, pats


def _dense_layer(g, case):
    d, qd, kd, F = case["d"], case["Hq"] * case["dh"], case["Hk"] * case["dh"], case["F"]
    w = {"Wq": g.normal((qd, d), d ** -0.5), "Wk": g.normal((kd, d), d ** -0.5), "Wv": g.normal((kd, d), d ** -0.5),
         "Wo": g.normal((qd, d), qd ** -0.5), "W1": g.normal((F, d), d ** -0.5), "W2": g.normal((F, d), F ** -0.5)}
    for n, k in (("bq", qd), ("bk", kd), ("bv", kd), ("bo", d), ("b1", F), ("b2", d)):
        w[n] = g.normal((k,), 0.02)
    for n in ("ln1", "ln2"):
        w[n + "_g"], w[n + "_b"] = g.normal((d,), 0.05, 1.0), g.normal((d,), 0.05)
    return w


def _desc(case, P, **kw):
    return sf.make_desc(case["B"], _length(case), case["d"], case["Hq"], case["Hk"], case["dh"], case["F"],
                        n_layers=case["nl"], P=P, dtype=_SF[case["dtype"]],
                        act=sf.SF_GELU_ERF if case.get("act") == "gelu" else sf.SF_RELU, c_factor=case["c"],
                        final_ln=case.get("final_ln", False), **kw)


def _fp8_codes(w, scale):
    return (w.float() / scale).clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8).contiguous()


def _prepare_encoder(case, seed, st):
    g = _Gen(seed, case["dtype"])
    pres, pid, pats = _inputs(case, seed, st)
    nl, L, B, d = case["nl"], _length(case), case["B"], case["d"]
    desc = st["desc"] = _desc(case, len(pats), n_sample=case["n_sample"])
    st["X"] = g.normal((B, L, d))
    st["dense"] = [_dense_layer(g, case) for _ in range(nl)]
    st["ln"] = {"g": g.normal((d,), 0.05, 1.0), "b": g.normal((d,), 0.05)} if case["final_ln"] else None
    st["gh"], st["gf"] = g.uniform((nl, len(pats), case["Hq"])), g.uniform((nl, len(pats), case["F"]))
    st["kh"], st["kf"] = [_keep(case["head_keep"], case["Hq"])] * nl, [_keep(case["ffn_keep"], case["F"])] * nl
    if case["n_sample"]:
        # one key sample per window, drawn with replacement from the whole sequence
        st["sample"] = torch.randint(0, L, (B, case["n_sample"]), generator=g.g, device="cuda", dtype=torch.int32)
    st["masks"] = sf.gate_scores_to_masks(desc, st["gh"], st["gf"], st["kh"], st["kf"])
    st["layers"] = [sf.compact_heads_channels(desc, l, st["dense"][l], st["masks"], st["kh"][l], st["kf"][l]) for l in range(nl)]
    if case["kind"] == "encoder":
        st["ws"] = sf.workspace(sf.encoder_workspace_bytes(desc, st["layers"]))
    elif case["kind"] == "fp8":
        # offline post-training quantisation: weights amax / 448, activations at about 5.5 standard deviations
        st["ffn8"], st["proj8"], act = [], [], 5.5 / 448.0
        for l, w in enumerate(st["dense"]):
            sc = {n: float(w[n].float().abs().max()) / 448.0 for n in ("W1", "W2", "Wo")}
            s_qkv = max(float(w[n].float().abs().max()) for n in ("Wq", "Wk", "Wv")) / 448.0
            d8 = dict(w, W1=_fp8_codes(w["W1"], sc["W1"]), W2=_fp8_codes(w["W2"], sc["W2"]), Wo=_fp8_codes(w["Wo"], sc["Wo"]),
                      **{n: _fp8_codes(w[n], s_qkv) for n in ("Wq", "Wk", "Wv")})
            st["ffn8"].append(sf.compact_ffn_fp8(desc, l, d8, sc, st["masks"], st["kf"][l], act, act))
            st["proj8"].append(sf.compact_proj_fp8(desc, l, d8, s_qkv, sc["Wo"], st["masks"], st["kh"][l], act, act))
        st["ws"] = sf.workspace(sf.encoder_fp8_workspace_bytes(desc, st["layers"]))
    else:
        # packed: the loader knows the presence masks, so it sizes the packed buffers for this batch
        seg = _segments(case)
        lens = [case["fusion"] + sum(n for n, p in zip(seg, row) if p) for row in pres.tolist()]
        runs = {}
        for p, n in zip(pid.tolist(), lens):
            runs[p] = runs.get(p, 0) + n
        Tc = sum(-(-n // 256) * 256 for n in runs.values()) + -(-L // 256) * 256
        st["tok_plan"] = sf.TokenPackPlan(B, L, Tc, "cuda")
        st["desc_p"] = _desc(case, len(pats), U_override=max(_active(n, case["c"]) for n in lens))
        st["ws"] = sf.workspace(sf.encoder_packed_workspace_bytes(st["desc_p"], st["layers"], Tc))


def _prepare_gqa(case, seed, st):
    g = _Gen(seed, case["dtype"])
    _inputs(case, seed, st)
    st["pid"] = None                          # one head map, whatever is missing
    B, L, nH, nG, dh = case["B"], _length(case), case["nH"], case["nG"], case["dh"]
    st["desc"] = sf.make_desc(B, L, nH * dh, nH, nG, dh, 64, dtype=_SF[case["dtype"]], c_factor=case["c"],
                              U_override=L if case["dense"] else -1)
    st["Q"], st["K"], st["V"] = (g.normal((B, n, L, dh)) for n in (nH, nG, nG))
    st["hg"] = torch.arange(nH, dtype=torch.int32, device="cuda").div(nH // nG, rounding_mode="floor").to(torch.int32).reshape(1, nH)
    st["ws"] = sf.workspace(sf.sparse_gqa_workspace_bytes(st["desc"], nH, nG))


def _prepare_moe(case, seed, st):
    g = _Gen(seed, case["dtype"])
    _, _, pats = _inputs(case, seed, st)
    E, P, d, F, B, L = case["experts"], len(pats), case["d"], case["F"], case["B"], _length(case)
    dt = _SF[case["dtype"]]
    kf = [_keep(0.4 + 0.4 * e / max(1, E - 1), F) for e in range(E)]      # ragged experts, 40 to 80 % kept
    dense = {"Wr": g.normal((E, d), d ** -0.5), "br": g.normal((E,), 0.02), "W1": g.normal((E, F, d), d ** -0.5),
             "b1": g.normal((E, F), 0.02), "W2": g.normal((E, F, d), F ** -0.5), "b2": g.normal((E, d), 0.02),
             "ln_g": g.normal((d,), 0.05, 1.0), "ln_b": g.normal((d,), 0.05)}
    masks = sf.gate_scores_to_masks(sf.make_desc(B, L, d, 8, 2, 8, F, n_layers=E, P=P, dtype=dt), g.uniform((E, P, 8)),
                                    g.uniform((E, P, F)), [1] * E, kf)
    st["desc"] = sf.make_desc(B, L, d, 8, 2, 8, F, n_layers=1, P=P, dtype=dt)
    st["moe"] = sf.compact_moe_experts(st["desc"], dense, masks["ffn_idx"], case["top_k"], kf)
    st["X"] = g.normal((B * L, d))
    st["ws"] = sf.workspace(sf.moe_ffn_workspace_bytes(st["desc"], st["moe"]))


def _prepare_gate(case, seed, st):
    g = _Gen(seed, case["dtype"])
    _, _, pats = _inputs(case, seed, st)
    nl, n, Hd, M = case["nl"], case["Hq"] + case["F"], case["hidden"], len(_segments(case))
    st["desc"] = _desc(case, len(pats))
    f = torch.float32
    st["gate"] = {"Wa": g.normal((nl, Hd, M), dtype=f), "ba": g.normal((nl, Hd), 0.3, dtype=f),
                  "Wb": g.normal((nl, n, Hd), Hd ** -0.5, dtype=f), "cb": g.normal((nl, n), 0.2, dtype=f),
                  "zeta": g.normal((nl, n), dtype=f), "gamma": g.uniform((nl,)).mul_(1.5).add_(0.5)}
    L, d, dh, U = _length(case), case["d"], case["dh"], _active(_length(case), case["c"])
    # multiply-adds times two of one kept head, K/V group and channel: the budget is a share of the dense network's
    st["cost"] = [2 * L * d * dh * 2 + 2 * L * L * dh + 4 * U * L * dh] * nl, [2 * L * d * dh * 2] * nl, [4 * L * d] * nl
    st["budget"] = int(case["budget"] * nl * (case["Hq"] * st["cost"][0][0] + case["Hk"] * st["cost"][1][0] + case["F"] * st["cost"][2][0]))


_PREPARE = {"encoder": _prepare_encoder, "fp8": _prepare_encoder, "packed": _prepare_encoder, "gqa": _prepare_gqa,
            "moe": _prepare_moe, "gate": _prepare_gate}


def prepare(case, seed):
    st = {"case": case}
    with sf.use_half("f16" if case["dtype"] == "f16" else "bf16"):
        _PREPARE[case["kind"]](case, seed, st)
    return st


# ------------------------------------------------------------------------------------------------ one pass
def _build_plan(st, out):
    """Keep masks and compacted weights; the tensors of the plan go into `out`."""
    sf.gate_scores_to_masks(st["desc"], st["gh"], st["gf"], st["kh"], st["kf"], out=st["masks"])
    for l, w in enumerate(st["dense"]):
        sf.compact_heads_channels(st["desc"], l, w, st["masks"], st["kh"][l], st["kf"][l], out=st["layers"][l])
    out.update((k, st["masks"][k]) for k in ("head_idx", "ffn_idx", "head_group"))
    for l, c in enumerate(st["layers"]):
        out.update(("%s_%d" % (n, l), getattr(c, n)) for n in ("Wqkv", "bqkv", "WoT", "W1", "b1", "W2T"))


def _run(case, st):
    kind, out = case["kind"], {}
    if kind == "moe":
        return {"Y": sf.moe_ffn_forward(st["desc"], st["moe"], st["X"], st["pid"], ws=st["ws"])}
    if kind == "gate":
        g_head, g_ffn = sf.gate_eval(st["desc"], st["gate"], st["patterns"])
        found = sf.budget_search(st["desc"], g_head, g_ffn, st["desc"].P - 1, *st["cost"], 0, st["budget"])
        masks = sf.gate_scores_to_masks(st["desc"], g_head, g_ffn, found["k_head"].tolist(), found["k_ffn"].tolist())
        return dict(masks, g_head=g_head, g_ffn=g_ffn, **found)
    # the allowed keys of this batch; none are masked when no sensor can be missing
    kv = sf.presence_to_key_valid(st["presence"], st["tok"]) if case["max_drop"] or kind == "packed" else None
    if kind == "gqa":
        out["O"] = sf.sparse_gqa_forward(st["desc"], st["Q"], st["K"], st["V"], st["hg"], None, kv, want_sel=False, ws=st["ws"])[0]
    elif kind == "fp8":
        out["Y"] = sf.encoder_forward_fp8(st["desc"], st["layers"], st["X"], st["ffn8"], st["proj8"], st["pid"], kv, st["ln"],
                                          ws=st["ws"])[0]
    elif kind == "packed":
        Xp, tp = sf.token_pack(st["desc"], st["X"], kv, st["pid"], plan=st["tok_plan"])
        Yp = sf.encoder_forward_packed(st["desc_p"], st["layers"], Xp, tp, st["pid"], st["ln"], ws=st["ws"])[0]
        out["Y"] = sf.token_unpack(st["desc"], Yp, tp)
    else:
        if case["plan"]:
            _build_plan(st, out)
        out["Y"] = sf.encoder_forward(st["desc"], st["layers"], st["X"], st["pid"], kv, st["ln"], ws=st["ws"],
                                      sample_idx=st.get("sample"))[0]
    return out


def run(state):
    case = state["case"]
    if case["dtype"] == "f16":
        with sf.use_half("f16"):
            return _run(case, state)
    return _run(case, state)


# ------------------------------------------------------------------------------------------------ what it cannot do without
def work(case):
    B, L, es = case["B"], _length(case), 4 if case["dtype"] == "f32" else 2
    P = len(_patterns(len(_segments(case)), case["max_drop"]))
    n1, n2 = _mean_allowed(case)
    kind = case["kind"]
    if kind == "gqa":
        nH, nG, dh = case["nH"], case["nG"], case["dh"]
        U = L if case["dense"] else _active(L, case["c"])
        rows = n1 * min(1.0, U / L) if case["dense"] else U           # queries of missing sensors are never active
        fl = B * nH * 4 * dh * (n2 if case["dense"] else rows * n1) + (0 if case["dense"] else B * nH * 2 * dh * n2)
        return {"bytes": B * L * dh * (2 * nH + 2 * nG) * es, "flops": fl}
    if kind == "moe":
        d, F, E, k = case["d"], case["F"], case["experts"], case["top_k"]
        kept = sum(_keep(0.4 + 0.4 * e / max(1, E - 1), F) for e in range(E))
        return {"bytes": 2 * B * L * d * es + P * 2 * kept * d * es, "flops": B * L * (k * 4 * d * kept / E + 2 * d * E)}
    d, Hq, Hk, dh, F, nl = (case[n] for n in ("d", "Hq", "Hk", "dh", "F", "nl"))
    if kind == "gate":
        n = (Hq + F) * nl
        return {"bytes": n * (4 * (case["hidden"] + 2) + 9 * P),        # parameters; score, mask and index of every unit
                "flops": n * P * case["hidden"] * 2.0}
    kh, kf, U = _keep(case["head_keep"], Hq), _keep(case["ffn_keep"], F), _active(L, case["c"])
    rows = n1 if kind == "packed" else L      # a masked batch still carries the tokens of missing sensors
    groups = min(Hk, kh)
    proj = 2 * d * dh * (kh + 2 * groups) * rows + 2 * min(rows, kh * U + 1) * kh * dh * d
    if case["n_sample"]:
        score = kh * 2 * n1 * case["n_sample"] * n1 / L * dh
    else:
        score = kh * 2 * n2 * dh if U < L else 0
    fl = B * nl * (proj + score + kh * 4 * min(U, n1) * n1 * dh + 4 * d * kf * rows)
    weights = P * nl * ((2 * kh + 2 * Hk) * dh + 2 * kf) * d
    by = 2 * B * L * d * es + weights * (1 if kind == "fp8" else es)
    if case.get("plan"):
        by += weights * es * 2                # the kept rows are read and written once more
    return {"bytes": by, "flops": fl}


def tolerance(case):
    """About four times what the same call shows with its sums in another order (features, channels or keys permuted).

    A 16-bit encoder decides on scores that carry the rounding of its Q and K: a query at the edge of the top-U set may be
    picked or not, which changes that row of one head (`max`); with every layer more rows carry such a change.  The FP8 codes
    are decisions of the same sort, and so is the routing of a token between two experts of almost equal logit.
    """
    kind, deep = case["kind"], case.get("nl", 1) > 1
    if kind == "gate":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 3e-5}
    f16 = case["dtype"] == "f16"
    if kind == "gqa":
        return {"rel": 2e-3 if f16 else 1.1e-2, "max": 0.02 if f16 else 0.1}
    if kind == "moe":
        return {"rel": 1e-3, "max": 0.5}
    if kind == "fp8":
        return {"rel": 1.1e-2, "max": 0.5}
    return {"rel": (4e-3 if deep else 1e-3) if f16 else (1.5e-2 if deep else 3e-3), "max": 0.5}
