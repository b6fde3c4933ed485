"""What the speed of this library is judged by: the passes a user's program makes through the binding.

A case is one pass over synthetic inputs that are already on the GPU, of one of four kinds:

  forward  route + forward, nothing kept for a backward pass; with "block" the normalisation in front of the
           router and the residual add of a transformer block (serving: decode batches, prompts, whole sequences)
  train    route + forward + backward: dX, router gradients and all three weight gradients of every expert; with
           "block" also the normalisation and its backward
  merge    the elementwise merge of N models' shared parameters (mean, or a weighted sum)
  adamw    the fused optimizer step on a stack of expert weights

Shapes: the seed model's feed-forward is d x 2.6875 d (4096 x 11008, or a smaller model of the same proportions),
C chunks per feed-forward give experts of width f / C ("split"), T is the number of tokens of the batch.
Buffers that a program keeps between calls (outputs, saved activations, workspace) are allocated in prepare().
"""
import math

import torch

from paper_2403_07816_amd import binding as B
from paper_2403_07816_amd import synth

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
MODES = {"topk": B.BTX_ROUTE_TOPK_RENORM, "switch": B.BTX_ROUTE_SWITCH_TOP1, "sample": B.BTX_ROUTE_SAMPLE_TOP1,
         "gumbel": B.BTX_ROUTE_GUMBEL_TOP1}
ALPHA = 0.01        # weight of the load-balancing loss
TAU = 0.5           # temperature of the Gumbel samples
EPS = 1e-5          # of the normalisation


def layer(kind, T, d, f, E, k, dtype="bf16", mode="topk", bias=0.0, cf=0.0, block=False):
    """bias: added to the router's logit of expert 0 (an overloaded expert); cf: capacity factor (0: nothing dropped)."""
    return dict(kind=kind, T=T, d=d, f=f, E=E, k=k, dtype=dtype, mode=mode, bias=bias, cf=cf, block=block)


def listed():
    cases = {
        # fp32 forward of a toy layer (unit tests, debugging, gradient checks of a new model): launches and host time
        "forward_toy_f32": layer("forward", 512, 64, 176, 4, 2, "f32"),
        # one decoding step of 16 sequences through the 7B-shaped layer inside its block: every expert's weights are
        # read for a handful of rows each
        "decode_16_bf16": layer("forward", 16, 4096, 11008, 4, 2, block=True),
        # a short prompt (or a speculative / chunked batch): about 150 rows per expert, a ragged count
        "prompt_301_bf16": layer("forward", 301, 4096, 11008, 4, 2, block=True),
        # one whole sequence, forward only
        "sequence_4096_bf16": layer("forward", 4096, 4096, 11008, 4, 2),
        # the MoE-finetuning step: 4 sequences, top-2, balanced experts
        "train_top2_bf16": layer("train", 16384, 4096, 11008, 4, 2),
        # top-1 sampled routing with one overloaded expert
        "train_sample_bf16": layer("train", 16384, 4096, 11008, 4, 1, mode="sample", bias=2.0),
        # every feed-forward split into 8 chunks: 32 experts of width 1376, top-8
        "train_split8_bf16": layer("train", 16384, 4096, 1376, 32, 8),
        # split into 16: 64 experts of width 688, which is no multiple of 32; a ragged batch
        "train_split16_bf16": layer("train", 1501, 4096, 688, 64, 8),
        # a smaller model of the same proportions, the whole block with its normalisation, a ragged batch
        "train_block_bf16": layer("train", 4001, 2048, 5504, 8, 2, block=True),
        # fp32 training of a small model (the reference run of a numerics question)
        "train_small_f32": layer("train", 2003, 512, 1376, 8, 2, "f32"),
        # the shared parameters of four 7B models averaged: 32 x 4 attention matrices and the embeddings
        "merge_mean_7b_bf16": dict(kind="merge", n=4, numel=128 * 4096 * 4096 + 32000 * 4096, dtype="bf16", weighted=False),
        # the optimizer step on the expert stack of the 7B-shaped layer, bf16 gradients and working copy
        "adamw_experts_bf16": dict(kind="adamw", numel=4 * 3 * 4096 * 11008, dtype="bf16", lowp=True),
    }
    return [dict(name=name, **case) for name, case in cases.items()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges the listed ones stand for; never more work than the listed one of its kind."""
    what = rng.choice(["serve", "serve", "train", "train", "train_odd", "train_f32", "forward_f32", "merge", "adamw"])
    if what in ("merge", "adamw"):
        dtype = rng.choice(["bf16", "bf16", "f32"])
        if what == "merge":
            n = rng.choice([2, 3, 4, 5, 7])
            most = (128 * 4096 * 4096 + 32000 * 4096) * 5 // (n + 1) // (2 if dtype == "f32" else 1)
            return dict(kind="merge", n=n, numel=_log_int(rng, 1 << 16, most), dtype=dtype, weighted=rng.random() < 0.3)
        return dict(kind="adamw", numel=_log_int(rng, 1 << 16, 4 * 3 * 4096 * 11008), dtype=dtype, lowp=rng.random() < 0.7)
    if what in ("train_f32", "forward_f32"):
        d, f = 8 * rng.randint(8, 64), 8 * rng.randint(8, 172)
        E = rng.choice([2, 4, 5, 8])
        kind = "train" if what == "train_f32" else "forward"
        return layer(kind, _log_int(rng, 16, 2003), d, f, E, 2, "f32", block=rng.random() < 0.3)
    if what == "train_odd":             # widths that are multiples of 8 but not of 32
        d, f = 32 * rng.randint(8, 127) + 8 * rng.randint(0, 3), 32 * rng.randint(4, 20) + 8 * rng.randint(1, 3)
        E = rng.choice([4, 8, 16, 64])
        return layer("train", _log_int(rng, 64, 1501), d, f, E, min(E // 2, rng.choice([2, 4, 8])))
    d = rng.choice([1024, 2048, 4096, 4096])
    split = rng.choice([1, 1, 2, 4, 8])
    n_ff = rng.choice([4, 4, 8]) if d < 4096 else 4
    E, f = n_ff * split, d * 43 // 16 // split
    mode, cf, bias = "topk", 0.0, 0.0
    k = min(2 * split, 8)
    if split == 1 and rng.random() < 0.4:
        mode, k, bias = rng.choice(["switch", "sample", "gumbel"]), 1, rng.choice([0.0, 2.0])
        cf = rng.choice([0.0, 1.5]) if mode == "switch" else 0.0
    if what == "serve":
        return layer("forward", _log_int(rng, 1, 4096), d, f, E, k, mode=mode, bias=bias, cf=cf, block=rng.random() < 0.5)
    most = 16384 if f % 32 == 0 else 1501 * 8 * 4096 * 688 // (k * d * f)
    return layer("train", _log_int(rng, 256, most), d, f, E, k, mode=mode, bias=bias, cf=cf, block=rng.random() < 0.3)


# ---- the state a program holds, one pass over it -------------------------------------------------------------


def _generator(seed, stream):
    return torch.Generator(device="cuda").manual_seed(seed * 7919 + stream)


def _prepare_layer(c, seed):
    T, d, f, E, k = c["T"], c["d"], c["f"], c["E"], c["k"]
    dtype, train = DTYPES[c["dtype"]], c["kind"] == "train"
    code = B.BTX_BF16 if c["dtype"] == "bf16" else B.BTX_F32
    L = synth.make_layer(T, d, f, E, dtype=dtype, seed=synth.BASE_SEED + seed, device="cuda", unit_rms=True,
                         router_bias=[c["bias"]] + [0.0] * (E - 1) if c["bias"] else None, with_dY=train,
                         with_U=c["mode"] == "sample", with_gumbel=c["mode"] == "gumbel")
    lib = B.load_library()
    ws = [lib.btx_moe_route_workspace_bytes(T, d, E, k), lib.btx_moe_ff_forward_workspace_bytes(T, d, f, E, k, code)]
    s = dict(case=c, L=L, routing=B.alloc_routing(T, E, k, "cuda"), out=torch.empty_like(L["x"]))
    if c["block"]:      # raw rows of varying length, a gain near one
        g = _generator(seed, 1)
        s["h"] = (L["x"].float() * torch.exp(0.5 * torch.randn((T, 1), generator=g, device="cuda"))).to(dtype)
        s["gain"] = 1.0 + 0.1 * torch.randn(d, generator=g, device="cuda")
        s["xn"], s["rstd"] = torch.empty_like(s["h"]), torch.empty(T, device="cuda")
    if train:
        ws.append(lib.btx_moe_ff_backward_workspace_bytes(T, d, f, E, k, code))
        s["saved"] = (torch.empty((T * k, f), dtype=dtype, device="cuda"), torch.empty((T * k, f), dtype=dtype, device="cuda"))
        s["grads"] = B.Grads(torch.empty_like(L["x"]), torch.empty((d, E), device="cuda"), torch.empty(E, device="cuda"),
                             torch.empty_like(L["W1"]), torch.empty_like(L["W3"]), torch.empty_like(L["W2"]))
        if c["block"]:
            ws.append(lib.btx_rmsnorm_backward_workspace_bytes(T, d))
            s["dH"], s["dgain"] = torch.empty_like(s["h"]), torch.empty(d, device="cuda")
    s["ws"] = torch.empty(max(ws), dtype=torch.uint8, device="cuda")
    return s


def _run_layer(s):
    c, L, r, ws, k = s["case"], s["L"], s["routing"], s["ws"], s["case"]["k"]
    mode, block, train = MODES[c["mode"]], c["block"], c["kind"] == "train"
    opts = dict(out=r, workspace=ws, tau=TAU, capacity_factor=c["cf"])
    if block:
        x, residual = s["xn"], s["h"]
        B.btx_moe_norm_route(s["h"], s["gain"], EPS, L["W_router"], L["b_router"], L["U"], k, mode, B.BTX_LB_TOKEN_FRAC,
                             ALPHA, xn=x, rstd=s["rstd"], **opts)
    else:
        x, residual = L["x"], None
        B.btx_moe_route(x, L["W_router"], L["b_router"], L["U"], k, mode, B.BTX_LB_TOKEN_FRAC, ALPHA, **opts)
    _, h1, h3 = B.btx_moe_ff_forward(x, L["W1"], L["W3"], L["W2"], r, save=train, out=s["out"], saved=s.get("saved"),
                                     workspace=ws, residual=residual)
    outputs = dict(out=s["out"], topk_idx=r.topk_idx, gates=r.gates, probs=r.probs, counts=r.counts, lb_loss=r.lb_loss)
    if not train:
        return outputs
    g = B.btx_moe_ff_backward(L["dY"], x, L["W_router"], L["W1"], L["W3"], L["W2"], r, h1, h3, mode, B.BTX_LB_TOKEN_FRAC,
                              ALPHA, 1.0, out=s["grads"], workspace=ws, noise=L["U"] if c["mode"] == "gumbel" else None,
                              tau=TAU)
    outputs.update(dX=g.dX, dW_router=g.dW_router, db_router=g.db_router, dW1=g.dW1, dW3=g.dW3, dW2=g.dW2)
    if block:
        dH, dgain = B.btx_rmsnorm_backward(g.dX, s["h"], s["gain"], s["rstd"], dres=L["dY"], dH=s["dH"], workspace=ws,
                                           dgain=s["dgain"])
        outputs.update(dH=dH, dgain=dgain)
    return outputs


def _prepare_merge(c, seed):
    base = torch.randn(c["numel"], generator=_generator(seed, 2), device="cuda") / 64.0
    copies = []
    for i in range(c["n"]):
        drift = torch.randn(c["numel"], generator=_generator(seed, 3 + i), device="cuda")
        copies.append(drift.mul_(0.1 / 64.0).add_(base).to(DTYPES[c["dtype"]]))
        del drift
    weights = [(i + 1) * 2.0 / (c["n"] * (c["n"] + 1)) for i in range(c["n"])] if c["weighted"] else None
    return dict(case=c, copies=copies, weights=weights, out=torch.empty_like(copies[0]))


def _run_merge(s):
    if s["weights"]:
        return B.btx_merge_weighted(s["copies"], s["weights"], out=s["out"])
    return B.btx_merge_average(s["copies"], out=s["out"])


def _prepare_adamw(c, seed):
    g, n = _generator(seed, 20), c["numel"]
    master = torch.randn(n, generator=g, device="cuda").div_(64.0)
    m = torch.randn(n, generator=g, device="cuda").mul_(1e-3)
    v = torch.randn(n, generator=g, device="cuda").square_().mul_(1e-6)
    grad = torch.randn(n, generator=g, device="cuda").mul_(1e-2).to(DTYPES[c["dtype"]])
    lowp = torch.empty(n, dtype=torch.bfloat16, device="cuda") if c["lowp"] else None
    return dict(case=c, master=master, m=m, v=v, grad=grad, lowp=lowp)


def _run_adamw(s):
    B.btx_adamw_step(s["master"], s["m"], s["v"], s["grad"], 100, 1e-4, weight_decay=0.1, lowp=s["lowp"])
    return [t for t in (s["master"], s["m"], s["v"], s["lowp"]) if t is not None]


def prepare(case, seed):
    c = dict(case)
    return {"merge": _prepare_merge, "adamw": _prepare_adamw}.get(c["kind"], _prepare_layer)(c, seed)


def run(state):
    return {"merge": _run_merge, "adamw": _run_adamw}.get(state["case"]["kind"], _run_layer)(state)


# ---- what a pass cannot do without, and how far another correct one may be off ------------------------------


def _rows(c):
    """Routed rows that the experts work on (the expected number where a capacity limit drops some)."""
    rows = c["T"] * c["k"]
    if c["cf"] > 0:
        share = math.exp(c["bias"]) / (math.exp(c["bias"]) + c["E"] - 1)      # of expert 0, roughly
        cap = math.ceil(c["cf"] * rows / c["E"])
        rest = (1.0 - share) / max(c["E"] - 1, 1)
        rows = int(min(rows * share, cap) + (c["E"] - 1) * min(rows * rest, cap))
    return rows


def work(case):
    c = case
    if c["kind"] == "merge":
        size = 2 if c["dtype"] == "bf16" else 4
        return {"bytes": (c["n"] + 1) * size * c["numel"], "flops": c["n"] * c["numel"]}
    if c["kind"] == "adamw":
        return {"bytes": (24 + (2 if c["dtype"] == "bf16" else 4) + (2 if c["lowp"] else 0)) * c["numel"],
                "flops": 16 * c["numel"]}
    T, d, f, E = c["T"], c["d"], c["f"], c["E"]
    size = 2 if c["dtype"] == "bf16" else 4
    rows = _rows(c)
    busy = E * (1.0 - (1.0 - 1.0 / E) ** rows)          # experts that receive a row, if all are equally likely
    weights, x = 3 * busy * d * f * size, T * d * size
    router = 4 * d * E + T * (8 * c["k"] + 4 * E)       # W_router in; indices, gates and probabilities out
    moved, flops = weights + 2 * x + router, 6 * rows * d * f + 2 * T * d * E
    if c["block"]:                                      # the normalised rows and the residual come from the same h
        flops += 4 * T * d
    if c["kind"] == "train":                            # x, dY, the weights in; dX and every weight gradient out; h1, h3 kept
        moved += 3 * E * d * f * size + weights + 3 * x + 8 * d * E + 4 * rows * f * size
        flops += 12 * rows * d * f + 4 * T * d * E
        if c["block"]:
            moved += 2 * x
            flops += 10 * T * d
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    c = case
    if c["kind"] == "merge":
        return "exact"      # the order of the sum and the one rounding are part of the entry points' description
    # The rest was measured against the same pass in fp64 (the routing's choices given): largest relative error seen,
    # times about four.
    if c["kind"] == "adamw":        # 4e-8; the working copy: single roundings to the other bf16 neighbour
        return {"rel": 1e-4, "max": 1e-2} if c["lowp"] else {"rel": 1e-6}
    # "differ": two sums of a logit in another order can order two experts differently whose logits agree to 1e-6
    if c["dtype"] == "f32":         # 7e-7; 4.5e-6 for the router's gradients, whose terms cancel
        return {"rel": 2e-5 if c["kind"] == "train" else 4e-6, "differ": 1e-3}
    # forward 2.9e-3; training 1.5e-2 to 2.3e-2 for the router's gradients (of experts that are nearly alike), 3.5e-3 else
    return {"rel": 3e-2 if c["kind"] == "train" else 1e-2, "max": 1.0 - 1e-9, "differ": 1e-3}
