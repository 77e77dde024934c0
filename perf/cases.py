"""The performance cases of the verify step: what a decoder that uses this library has it do.

Every case is one pass through the public entry points (``paper_2604_05650_amd.binding``), either
by its Python functions with nothing prepared (``api = "call"``: outputs and workspaces are
allocated inside, as a script or a test does it) or through the C ABI with argument structures and
workspaces a serving loop lays out once (``api = "args"``, as ``bench.py`` does it).

kind      one pass is
attn      lvspec_verify_attn over a stack of layers, one KV cache per layer
step      the same stack, then lvspec_visual_relevance and lvspec_loose_accept
rel       lvspec_visual_relevance
accept    lvspec_loose_accept
prefill   lvspec_hv_prepare
commit    lvspec_kv_commit of a draft tree, all layers of a cache in one call

Sizes: the benchmark's configurations (2048 to 65536 cached keys, hidden sizes 1024 to 8192, 8192
to 152064 vocabulary rows, one to four sequences), batches of sequences of unequal lengths as a
server holds them, draft chains of 1 to 16 tokens and trees of up to 32.
"""
from __future__ import annotations

import ctypes as C
import math

import torch

from paper_2604_05650_amd import binding as L
from paper_2604_05650_amd import synth

D = 128
DEV = "cuda:0"
MOST_BYTES = 6.0e9        # a drawn case moves no more than this
VOCAB = 152064

ATTN = dict(B=1, gamma=5, branches=1, Hq=40, Hkv=8, kv_lo=16384, kv_hi=16384, layers=1,
            host_len=True, extras=False, api="args")
HID = dict(d=5120, lv=14336, top_n=10, prepared=False)
ACC = dict(V=VOCAB, topk=4, bonus=False, rule=0, logits=False, entropy=False)


def listed():
    return [
        # the smallest step: one layer of a tiny target, called from Python (launches, host work)
        dict(name="tiny-step", kind="step", **{
            **ATTN, **HID, **ACC, "gamma": 4, "Hq": 8, "Hkv": 2, "kv_lo": 2048, "kv_hi": 2048,
            "d": 1024, "lv": 1568, "V": 8192, "api": "call"}),
        # the headline: one user's verify step at the 32B shape, 64 layers, five drafts
        dict(name="32b-step", kind="step", **{**ATTN, **HID, **ACC, "layers": 64}),
        # the same with a draft tree of two chains of ten tokens
        dict(name="32b-tree-step", kind="step", **{
            **ATTN, **HID, **ACC, "layers": 64, "gamma": 20, "branches": 2}),
        # layers of the 72B shape over a shorter video: a short stream per call
        dict(name="72b-layers", kind="attn", **{
            **ATTN, "Hq": 64, "kv_lo": 7296, "kv_hi": 7296, "layers": 16}),
        # long videos, four sequences, eight drafts at the 72B shape
        dict(name="long-video-step", kind="step", **{
            **ATTN, **HID, **ACC, "B": 4, "gamma": 8, "Hq": 64, "kv_lo": 65536, "kv_hi": 65536,
            "d": 8192, "lv": 63488}),
        # a server's batch: sequences between a short clip and a long one, lengths on the device
        dict(name="serve-ragged", kind="attn", **{
            **ATTN, "B": 16, "kv_lo": 2048, "kv_hi": 32768, "layers": 4, "host_len": False,
            "extras": True, "api": "call"}),
        # plain decoding of a larger batch: one row per sequence, lengths known to the host
        dict(name="decode-batch", kind="attn", **{
            **ATTN, "B": 24, "gamma": 1, "Hq": 28, "Hkv": 4, "kv_lo": 3000, "kv_hi": 9000,
            "layers": 8}),
        # relevance with the largest N of the sensitivity study
        dict(name="relevance-top100", kind="rel", **{**ATTN, **HID, "top_n": 100, "api": "call"}),
        # lm_head and acceptance for a batch, with the row after the last draft
        dict(name="accept-batch", kind="accept", **{
            **ATTN, **HID, **ACC, "B": 16, "bonus": True, "entropy": True}),
        # one sequence whose caller samples: logits, wide top-k, the entropy-gated rule
        dict(name="accept-logits", kind="accept", **{
            **ATTN, **HID, **ACC, "d": 3584, "topk": 16, "rule": 2, "logits": True,
            "entropy": True, "api": "call"}),
        # once per video at prefill: the inverse norms of its hidden states
        dict(name="prefill-norms", kind="prefill", **{
            **ATTN, **HID, "B": 2, "d": 8192, "lv": 6272, "api": "call"}),
        # a verified tree joins the caches of all layers
        dict(name="tree-commit", kind="commit", **{
            **ATTN, "gamma": 20, "branches": 2, "kv_lo": 4096, "kv_hi": 4096, "layers": 28,
            "api": "call"}),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attn"] * 7 + ["step"] * 4 + ["rel"] * 3 + ["accept"] * 4 +
                      ["prefill", "commit"])
    while True:
        c = dict(kind=kind, **ATTN)
        c["B"] = _log(rng, 1, 32)
        c["Hq"], c["Hkv"] = rng.choice([(8, 2), (28, 4), (40, 8), (64, 8)])
        c["kv_hi"] = _log(rng, 500, 65536)
        c["kv_lo"] = c["kv_hi"] if rng.random() < 0.4 else max(1, int(c["kv_hi"] * rng.uniform(0.05, 1)))
        if kind == "commit" or rng.random() < 0.25:
            c["branches"] = rng.choice([2, 2, 3])
            c["gamma"] = c["branches"] * rng.randint(2, 10)
        else:
            c["gamma"] = rng.randint(1, 16)
        c["host_len"] = rng.random() < 0.5
        c["extras"] = rng.random() < 0.3
        c["api"] = rng.choice(["args", "call"])
        if kind in ("attn", "step", "commit"):
            c["layers"] = rng.choice([1, 2, 4, 8, 16, 32])
        if kind in ("step", "rel", "accept", "prefill"):
            c.update(HID, d=rng.choice([1024, 2048, 3584, 4096, 5120, 8192]),
                     lv=c["kv_hi"] * 7 // 8 if kind == "step" else _log(rng, 200, 64000),
                     top_n=rng.choice([1, 5, 10, 10, 100]), prepared=rng.random() < 0.3)
        if kind in ("step", "accept"):
            c.update(ACC, V=rng.choice([8192, 32000, VOCAB, VOCAB]), topk=rng.choice([1, 4, 4, 16]),
                     bonus=rng.random() < 0.4 and kind == "accept", rule=rng.choice([0, 0, 1, 2]),
                     logits=rng.random() < 0.2, entropy=rng.random() < 0.4)
        w = work(c)
        held = c["layers"] * c["B"] * c["Hkv"] * _cap(c) * D * 4    # bytes of the caches themselves
        if 2e5 < w["bytes"] <= MOST_BYTES and (kind != "commit" or held <= MOST_BYTES):
            return c


def _lens(case):
    """Cached keys per sequence: spread evenly over the logarithm between the two ends."""
    B, lo, hi = case["B"], case["kv_lo"], case["kv_hi"]
    return [int(round(lo * (hi / lo) ** ((b + 0.5) / B))) for b in range(B)]


def _cap(case):
    return -(-(case["kv_hi"] + case["gamma"]) // 128) * 128


def work(case):
    k, B, g, lay = case["kind"], case["B"], case["gamma"], case["layers"]
    nbytes = flops = 0.0
    if k in ("attn", "step"):
        keys = sum(n + g for n in _lens(case)) * lay
        nbytes += keys * case["Hkv"] * D * 4 + 4.0 * lay * B * g * case["Hq"] * D
        flops += 4.0 * keys * g * case["Hq"] * D
    if k in ("rel", "step"):
        nbytes += 2.0 * B * (case["lv"] + g) * case["d"]
        flops += 2.0 * B * case["lv"] * g * case["d"]
    if k in ("accept", "step"):
        rows = B * (g + (case["branches"] if case["bonus"] else 0))
        nbytes += 2.0 * (case["V"] + rows) * case["d"] + (4.0 * rows * case["V"] if case["logits"] else 0)
        flops += 2.0 * rows * case["V"] * case["d"]
    if k == "prefill":
        nbytes += B * case["lv"] * (2.0 * case["d"] + 4)
        flops += 2.0 * B * case["lv"] * case["d"]
    if k == "commit":     # the accepted rows of half of the sequences, read and written
        nbytes += 4.0 * lay * B * (g // case["branches"]) * case["Hkv"] * D * 2 / 2
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # About four times what the same formulas in 64 bits showed.  Attention: bf16 probabilities and
    # a bf16 result (2.1e-3, largest single difference 7.9e-3); the rest holds 32-bit sums and whole
    # numbers that only a tie could move; probabilities pass on the absolute error of logits near
    # 10, summed in another order they moved by 6.1e-6.
    if case["kind"] == "commit":
        return "exact"
    if case["kind"] in ("attn", "step"):
        return {"rel": 8e-3, "max": 3.2e-2, "differ": 2e-3}
    return {"rel": 2.5e-5, "max": 1e-4, "differ": 2e-3}


def _normal(gen, shape, std):
    n = math.prod(shape)
    out = torch.empty((n,), dtype=torch.bfloat16, device=DEV)
    for s in range(0, n, 1 << 27):
        e = min(n, s + (1 << 27))
        out[s:e] = torch.randn((e - s,), generator=gen, device=DEV) * std
    return out.view(shape)


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(synth.BASE_SEED + int(seed))
    kind, B, g, br, lay = (case[x] for x in ("kind", "B", "gamma", "branches", "layers"))
    chain, chains = g // br, B * br
    s = {"case": case}
    lens = [_lens(case)[(b * 7 + int(seed)) % B if B % 7 else (b + int(seed)) % B] for b in range(B)]
    kv_len = torch.tensor(lens, dtype=torch.int32, device=DEV)
    if kind in ("attn", "step", "commit"):
        cap = _cap(case)
        s["k"] = _normal(gen, (lay, B, case["Hkv"], cap, D), 1.0)
        s["v"] = _normal(gen, (lay, B, case["Hkv"], cap, D), 1.0)
        s["kv_len"] = kv_len
    if kind in ("attn", "step"):
        s["q"] = _normal(gen, (lay, B, g, case["Hq"], D), 1.0)
        s["out"] = torch.empty_like(s["q"])
        s["opt"] = dict(
            vis_begin=torch.full_like(kv_len, 16),
            vis_end=torch.minimum(16 + kv_len * 7 // 8, kv_len),
            draft_mask=synth.branch_mask(br, chain) if br > 1 else None,
            kv_len_host=lens if case["host_len"] else None,
            max_kv_len=max(lens) if case["host_len"] else 0)
    if kind in ("rel", "step", "prefill"):
        s["h_v"] = _normal(gen, (B, case["lv"], case["d"]), 1.0)
        s["l_v"] = torch.full((B,), case["lv"], dtype=torch.int32, device=DEV)
        s["inv"] = L.hv_prepare(s["h_v"]) if case["prepared"] and kind != "prefill" else None
    if kind in ("rel", "accept", "step"):
        rows = chain + 1 if kind in ("accept", "step") and case["bonus"] else chain
        s["h_d"] = _normal(gen, (chains, rows, case["d"]), 1.0)
    if kind in ("rel", "step"):       # some drafts name what the video shows, some do not
        beta = torch.rand((B, g, 1), generator=gen, device=DEV)
        row = torch.randint(case["lv"], (B, g), generator=gen, device=DEV)
        seen = torch.stack([s["h_v"][b, row[b]] for b in range(B)]).float()
        s["h_d"] = (s["h_d"].view(B, g, case["d"]).float() + beta * seen).to(torch.bfloat16)
        s["h_d"] = s["h_d"].view(chains, chain, case["d"])
    if kind in ("accept", "step"):
        s["w"] = _normal(gen, (case["V"], case["d"]), 0.02)
        ids = torch.randint(case["V"], (chains, s["h_d"].shape[1]), generator=gen, device=DEV)
        # most drafts are what the target says (its row leans towards that token), some are not
        lean = 300.0 / case["d"] ** 0.5          # that token's logit: six standard deviations
        s["h_d"] = (s["h_d"].float() + lean * s["w"][ids].float()).to(torch.bfloat16)
        keep = torch.rand(ids.shape, generator=gen, device=DEV) < 0.7
        other = torch.randint(case["V"], ids.shape, generator=gen, device=DEV)
        s["draft"] = torch.where(keep, ids, other)[:, :chain].to(torch.int32).contiguous()
        s["relevance"] = torch.rand((B, g), generator=gen, device=DEV)
        s["acc"] = dict(topk=case["topk"], n_branches=br, bonus_row=case["bonus"], rule=case["rule"],
                        entropy_threshold=0.2 if case["rule"] else 0.0,
                        defer_window=4 if case["rule"] == 2 else 0)
        s["n_loose"] = L.n_loose(0.7, chain)
    if kind == "commit":
        s["accept_len"] = torch.randint(1, chain + 1, (chains,), generator=gen, device=DEV, dtype=torch.int32)
        s["best"] = torch.randint(br, (B,), generator=gen, device=DEV, dtype=torch.int32)
    if case["api"] == "args":
        _lay_out(s)
    return s


def _space(nbytes):
    return torch.empty((max(256, int(nbytes)),), dtype=torch.uint8, device=DEV)


def _lay_out(s):
    """Argument structures, outputs and workspaces of a loop that calls the C ABI."""
    case, lib = s["case"], L.raw()
    kind, B, g, br = case["kind"], case["B"], case["gamma"], case["branches"]
    calls, keep = [], []
    if kind in ("attn", "step"):
        shape = (case["layers"], B, case["Hq"], g)
        s["lse"] = torch.empty(shape, device=DEV) if case["extras"] else None
        s["mass"] = torch.empty(shape, device=DEV) if case["extras"] else None
        for i in range(case["layers"]):
            a = L.verify_attn_args(s["q"][i], s["k"][i], s["v"][i], s["kv_len"], out=s["out"][i],
                                   lse=s["lse"][i] if case["extras"] else None,
                                   vis_mass=s["mass"][i] if case["extras"] else None, **s["opt"])
            if not keep:
                keep.append(_space(lib.lvspec_verify_attn_workspace(C.byref(a))))
            a.workspace, a.workspace_bytes = keep[0].data_ptr(), keep[0].numel()
            calls.append((lib.lvspec_verify_attn, a))
    if kind in ("rel", "step"):
        s["relevance"] = torch.empty((B, g), device=DEV)
        a = L.visual_relevance_args(s["h_d"].view(B, g, case["d"]), s["h_v"], s["l_v"], case["top_n"],
                                    relevance=s["relevance"], hv_inv_norm=s["inv"])
        keep.append(_space(lib.lvspec_visual_relevance_workspace(C.byref(a))))
        a.workspace, a.workspace_bytes = keep[-1].data_ptr(), keep[-1].numel()
        calls.append((lib.lvspec_visual_relevance, a))
    if kind in ("accept", "step"):
        s["outs"] = L.alloc_accept_outputs(B * br, g // br, case["V"], case["topk"], DEV, case["logits"],
                                           n_branches=br, return_entropy=case["entropy"],
                                           bonus_row=case["bonus"])
        a = L.loose_accept_args(s["h_d"], s["w"], s["draft"], s["relevance"].view(B * br, -1),
                                s["n_loose"], g // br, loose_topk_gate=0, outs=s["outs"], **s["acc"])
        keep.append(_space(lib.lvspec_loose_accept_workspace(C.byref(a))))
        a.workspace, a.workspace_bytes = keep[-1].data_ptr(), keep[-1].numel()
        calls.append((lib.lvspec_loose_accept, a))
    s["calls"] = [(fn, C.byref(a)) for fn, a in calls]
    s["keep"] = keep


def run(s):
    case = s["case"]
    kind, B, g, br = case["kind"], case["B"], case["gamma"], case["branches"]
    if kind == "prefill":
        return L.hv_prepare(s["h_v"])
    if kind == "commit":
        new = L.kv_commit(s["k"], s["v"], s["kv_len"], s["accept_len"], g // br,
                          best_branch=s["best"], n_branches=br)
        return {"k": s["k"], "v": s["v"], "new_len": new}
    if case["api"] == "args":
        stream = torch.cuda.current_stream().cuda_stream
        for fn, a in s["calls"]:
            rc = fn(a, stream)
            if rc != L.OK:
                raise L.LvspecError(rc)
        return {x: s[x] for x in ("out", "lse", "mass", "relevance", "outs") if s.get(x) is not None}
    r = {}
    if kind in ("attn", "step"):
        for i in range(case["layers"]):
            got = L.verify_attn(s["q"][i], s["k"][i], s["v"][i], s["kv_len"], out=s["out"][i],
                                return_lse=case["extras"], return_vis_mass=case["extras"], **s["opt"])
            if case["extras"]:
                r[f"lse{i:02d}"] = got[1]
                if i == 0:
                    r["mass"] = got[2]
        r["out"] = s["out"]
    rel = s.get("relevance")
    if kind in ("rel", "step"):
        rel = L.visual_relevance(s["h_d"].view(B, g, case["d"]), s["h_v"], s["l_v"], case["top_n"],
                                 hv_inv_norm=s["inv"])
        r["relevance"] = rel
    if kind in ("accept", "step"):
        r["outs"] = L.loose_accept(s["h_d"], s["w"], s["draft"], rel.view(B * br, -1), s["n_loose"], g // br,
                                   return_logits=case["logits"], return_entropy=case["entropy"], **s["acc"])
    return r
