"""Workloads of the MoE-layer library for timing and for comparing two builds of it.

A case is a dict of sizes and options.  `prepare` makes what a training or inference program holds before the
call (weights, inputs, a MoELayer with its buffers), `run` is one pass through the public entry points, `work` the
bytes and operations that pass cannot do without, `tolerance` how far another correct implementation of the same
precision may be off.  `listed` are the named workloads, `draw` gives further ones of the same ranges.

Kinds:
  step      forward and backward of a MoELayer (all the library's calls of a training step)
  forward   forward only of a MoELayer that saves nothing for a backward (evaluation, generation)
  mx8       expert forward on 8-bit block-scaled operands: quantise the layer input, the two products, combine
  dispatch  route, copy the rows into expert order, combine them again: what surrounds an expert-parallel exchange
"""
import math

import torch

from paper_2508_02317_amd import libmoe as L
from paper_2508_02317_amd.layer import MoELayer

_WEIGHT_STD = 0.02                       # router and expert weights
_LONG = dict(T=40960, d=2048, E=128, k=8, f=768)


def _case(kind, T, d, E, k, f, dtype="bf16", **options):
    c = dict(kind=kind, T=T, d=d, E=E, k=k, f=f, dtype=dtype, renorm=1, gather=True, save_gu=True, router=False,
             prerouted=False, mixed=False)
    c.update(options)
    return c


def listed():
    a3b = dict(d=2048, E=128, k=8, f=768)          # the 30B-A3B-class layer
    cases = {
        # the small full-precision layer of the parity configuration: launches and host time
        "tiny_f32_step": _case("step", 256, 128, 8, 2, 256, dtype="f32"),
        # few, wide experts: a small bf16 training step
        "small_step": _case("step", 4096, 1024, 16, 2, 2048),
        # one 8K-token micro-batch of the 30B-A3B-class layer
        "a3b_8k_step": _case("step", 8192, **a3b),
        # the same through MoELayer's default call sequence: expert-ordered copies written, combine backward separate
        "a3b_8k_separate_step": _case("step", 8192, **a3b, gather=False),
        # one expert-parallel rank: 16 local experts, rows already routed, two thirds of them on one expert
        "a3b_ep_skew_step": _case("step", 16384, 2048, 16, 1, 768, prerouted=True),
        # one sequence shard of a 160K-token multimodal sequence, text and patch rows of different scale
        "a3b_long_step": _case("step", mixed=True, **_LONG),
        # an odd last micro-batch from hidden states: router linear in the step, pre-activations recomputed
        "a3b_odd_router_step": _case("step", 1531, **a3b, router=True, save_gu=False),
        # one generation step of a small batch: a row or so per expert
        "a3b_few_tokens_forward": _case("forward", 16, **a3b, save_gu=False),
        # evaluation of one short document, selection weights not renormalised
        "a3b_2k_forward": _case("forward", 2047, **a3b, save_gu=False, renorm=0),
        # expert forward of the 8K micro-batch with 8-bit operands
        "a3b_8k_mx8_forward": _case("mx8", 8192, **a3b),
        # routing and row movement of an expert-parallel rank's 16K tokens over all 128 experts
        "a3b_16k_dispatch": _case("dispatch", 16384, **a3b),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _log_int(rng, lo, hi, multiple=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(multiple, int(round(v / multiple)) * multiple)


def draw(rng):
    kind = rng.choice(["step", "step", "step", "router", "ep", "forward", "forward", "mx8", "dispatch", "f32"])
    if kind == "f32":
        return _case("step", _log_int(rng, 16, 1024), _log_int(rng, 64, 512, 8), rng.choice([4, 8, 16, 24]), rng.randint(1, 4),
                     _log_int(rng, 64, 512, 8), dtype="f32", gather=rng.random() < 0.7, save_gu=rng.random() < 0.7, renorm=rng.randint(0, 1))
    multiple = 128 if kind == "mx8" else rng.choice([64, 64, 64, 8])     # widths are multiples of 64, now and then only of 8
    d, f = _log_int(rng, 512, 4096, multiple), _log_int(rng, 256, 3072, multiple)
    E, k = rng.choice([8, 16, 32, 60, 64, 128]), rng.choice([1, 2, 4, 6, 8])
    T = _log_int(rng, 1, 512) if kind == "forward" and rng.random() < 0.6 else _log_int(rng, 128, 40960)
    options = {}
    if kind == "ep":
        E, k, options = rng.choice([8, 16, 32]), 1, dict(prerouted=True)
    if kind == "router":
        E, options = rng.choice([8, 16, 32, 64, 128]), dict(router=True)
    if kind in ("step", "ep", "router"):
        options.update(gather=rng.random() < 0.7, save_gu=rng.random() < 0.7, mixed=rng.random() < 0.3)
    if kind == "forward":
        options.update(save_gu=False)
    if kind != "ep" and kind != "mx8":
        options.update(renorm=int(rng.random() < 0.7))
    # no more weights and no more arithmetic than the largest listed case
    top = float(_LONG["d"]) * _LONG["f"]
    E = max(k, min(E, int(_LONG["E"] * top / (d * f)) // 8 * 8)) if d * f * E > _LONG["E"] * top else E
    T = max(1, min(T, int(_LONG["T"] * _LONG["k"] * top / (k * d * f)), int(_LONG["T"] * _LONG["k"] * _LONG["d"] / (k * d))))
    return _case("step" if kind in ("router", "ep") else kind, T, d, E, k, f, **options)


def _normal(gen, shape, std, dtype):
    """N(0, std) rounded to dtype, drawn slab by slab so that no fp32 copy of a large weight exists."""
    out = torch.empty(shape, dtype=dtype, device="cuda")
    flat, step = out.view(-1), 1 << 26
    for s in range(0, flat.numel(), step):
        part = flat[s:s + step]
        part.copy_(torch.randn(part.numel(), generator=gen, device="cuda").mul_(std))
    return out


def _modality_scale(gen, T):
    """Alternating runs of text rows (1) and patch rows (4), 64 to 2048 rows long."""
    runs = torch.randint(64, 2049, (T // 64 + 2,), generator=gen, device="cuda").cumsum(0)
    run_of_row = torch.searchsorted(runs, torch.arange(T, device="cuda"), right=True)
    return 1.0 + 3.0 * (run_of_row % 2).float()


def _local_share(gen, T, E):
    """Rows an expert-parallel exchange has delivered to one of 8 ranks: local expert and combine weight of each row,
    from top-8 routing over 8 E experts whose popularity falls off as a Zipf law (exponent 1.2)."""
    EG, kG, tok = 8 * E, 8, 2 * T + 64
    e = torch.arange(EG, device="cuda")
    rank = (e % E) * 8 + e // E + 1
    z = torch.randn(tok, EG, generator=gen, device="cuda") * 0.9 - 1.2 * torch.log(rank.float())
    top, idx = torch.topk(z, kG, dim=1)
    w = torch.softmax(top, dim=1)
    keep = (idx < E).view(-1).nonzero().view(-1)[:T]
    keep = keep.repeat(-(-T // keep.numel()))[:T]
    return idx.view(-1)[keep].to(torch.int32).view(T, 1).contiguous(), w.view(-1)[keep].view(T, 1).contiguous()


def prepare(case, seed):
    c = case
    T, d, E, k, f = c["T"], c["d"], c["E"], c["k"], c["f"]
    dtype = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    s = {"case": c}
    x = _normal(gen, (T, d), 1.0, dtype)
    if c["mixed"]:
        x = (x.float() * _modality_scale(gen, T)[:, None]).to(dtype)
    s["x"] = x
    w_router = _normal(gen, (E, d), _WEIGHT_STD, dtype)
    if c["prerouted"]:
        s["idx"], s["w"] = _local_share(gen, T, E)
    elif not c["router"]:
        s["logits"] = (x.float() @ w_router.float().t()).contiguous()
    if c["kind"] == "dispatch":
        i32 = lambda *n: torch.empty(n, dtype=torch.int32, device="cuda")
        s["route"] = (i32(T, k), torch.empty((T, k), device="cuda"), i32(E), i32(E + 1))
        s["rows"] = (torch.empty((T * k, d), dtype=dtype, device="cuda"), i32(T * k), i32(T * k))
        s["y"] = torch.empty((T, d), dtype=dtype, device="cuda")
        s["ws"] = torch.empty(max(L.lib.moe_route_topk_workspace_bytes(T, E, k), L.lib.moe_permute_workspace_bytes(T, E, k), 256),
                              dtype=torch.uint8, device="cuda")
        return s
    wg, wu, wd = (_normal(gen, n, _WEIGHT_STD, dtype) for n in ((E, f, d), (E, f, d), (E, d, f)))
    if c["kind"] == "mx8":
        s["weights"] = [L.moe_mx8_quantise(w) for w in (wg, wu, wd)]     # once per optimiser step
        s["xq"] = L.moe_mx8_quantise(x)
        s["topk_idx"], s["topk_w"], _, s["offsets"] = L.moe_route_topk(s["logits"], k, c["renorm"])
        _, s["row_of_pair"], s["pair_of_row"] = L.moe_permute(None, s["topk_idx"], s["offsets"], E)
        P = T * k
        s["out"] = (torch.empty((P, f), dtype=torch.uint8, device="cuda"), torch.empty((f // 128, P), dtype=torch.int32, device="cuda"),
                    torch.empty((P, d), dtype=dtype, device="cuda"))
        s["y"] = torch.empty((T, d), dtype=dtype, device="cuda")
        s["ws"] = torch.empty(L.lib.moe_grouped_gemm_swiglu_fwd_mx8_workspace_bytes(P, d, f, E), dtype=torch.uint8, device="cuda")
        return s
    s["layer"] = MoELayer(T, d, E, k, f, dtype, wg, wu, wd, renorm=c["renorm"], prerouted=c["prerouted"], save_gu=c["save_gu"],
                          w_router=w_router if c["router"] else None, gather=c["gather"])
    if c["kind"] == "step":
        s["dy"] = _normal(gen, (T, d), 1.0, dtype)
    return s


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "dispatch":
        idx, w, counts, offsets = L.moe_route_topk(s["logits"], c["k"], c["renorm"], out=s["route"], ws=s["ws"])
        xp, row_of_pair, pair_of_row = L.moe_permute(s["x"], idx, offsets, c["E"], out=s["rows"], ws=s["ws"])
        y = L.moe_unpermute_combine_fwd(xp, w, row_of_pair, c["T"], c["k"], out=s["y"])
        return {"y": y, "xp": xp, "row_of_pair": row_of_pair, "pair_of_row": pair_of_row, "topk_idx": idx, "topk_w": w,
                "counts": counts, "offsets": offsets}
    if c["kind"] == "mx8":
        (wgq, wgs), (wuq, wus), (wdq, wds) = s["weights"]
        xq, xs = L.moe_mx8_quantise(s["x"], out=s["xq"])
        _, _, yp = L.moe_grouped_gemm_swiglu_fwd_mx8(xq, xs, wgq, wgs, wuq, wus, wdq, wds, s["offsets"], pair_of_row=s["pair_of_row"],
                                                     k=c["k"], out=s["out"], ws=s["ws"])
        y = L.moe_unpermute_combine_fwd(yp, s["topk_w"], s["row_of_pair"], c["T"], c["k"], out=s["y"])
        return {"y": y, "yp": yp, "x_codes": xq, "x_scales": xs}
    layer = s["layer"]
    if c["prerouted"]:
        layer.forward(s["x"], topk_idx=s["idx"], topk_w=s["w"])
    else:
        layer.forward(s["x"], logits=s.get("logits"))
    out = {"y": layer.y, "topk_idx": layer.topk_idx, "topk_w": layer.topk_w, "counts": layer.counts}
    if c["kind"] == "step":
        layer.backward(s["dy"], logits=s.get("logits"))
        out.update(dx=layer.dx, dw_gate=layer.dw_gate, dw_up=layer.dw_up, dw_down=layer.dw_down)
        if not c["prerouted"]:
            out["dlogits"] = layer.dlogits
        if c["router"]:
            out["dw_router"] = layer.dw_router
    return out


def work(case):
    c = case
    T, d, E, k, f = (float(c[n]) for n in ("T", "d", "E", "k", "f"))
    P, es = T * k, 4.0 if c["dtype"] == "f32" else 2.0
    routing = T * E * 4 + P * 8                                 # logits in, expert and weight of every pair out
    if c["kind"] == "dispatch":
        return {"bytes": routing + P * 8 + T * d * es + 2 * P * d * es + T * d * es, "flops": 2 * P * d}
    used = E * (1.0 - (1.0 - k / E) ** T)                       # experts that have rows under near-uniform routing
    if c["kind"] == "mx8":
        weights = 3 * used * d * f * (1 + 1 / 32)
        return {"bytes": weights + 2 * T * d * es + P * d * es + T * d, "flops": 6 * P * d * f}
    router = (2 * T * d * E, E * d * es) if c["router"] else (0.0, 0.0)
    rows, weights = T * d * es, 3 * used * d * f * es
    if c["kind"] == "forward":
        return {"bytes": routing + 2 * rows + weights, "flops": 6 * P * d * f}
    grads = 3 * E * d * f * es                                  # experts without rows get zeros
    return {"bytes": (P * 8 if c["prerouted"] else 2 * routing) + 4 * rows + weights + grads + 2 * router[1],
            "flops": 18 * P * d * f + 3 * router[0]}


def tolerance(case):
    """About four times the largest errors seen against the same layer evaluated in 64 bits and between MoELayer's two call
    sequences, which sum and round in different places (T = 130..2048, E = 16 and 32, the widths of the listed cases)."""
    if case["dtype"] == "f32":               # seen: 8e-7 and 7e-6
        return {"rel": 3e-6, "max": 3e-5}
    if case["kind"] == "dispatch":           # fp32 weights to 5e-8; a weighted sum of equal rows may round to the neighbouring bf16 value
        return {"rel": 2e-4, "max": 1e-2}
    out = {"rel": 1.2e-2, "max": 0.3}        # seen: 2e-3 to 4.7e-3, and 0.02 to 0.09
    if case["router"]:                       # logits summed in another order may swap two experts that tie in fp32
        out["differ"] = 1e-3
    return out
