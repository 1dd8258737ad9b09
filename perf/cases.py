"""The calls whose speed is tracked: the layer, its training step and the encoder layers around it,
through the public entry points of ``paper_2006_16668_amd``, as a program that uses them calls them.

A case is a dict of plain values.  ``kind`` says which call it is:

  forward   moe_forward (``prepacked``: moe_forward_prepacked, gate weights packed once beforehand)
  train     moe_forward_train + moe_backward
  attention moe_self_attention
  encoder   moe_encoder_pair_forward_train + moe_encoder_pair_backward

and the rest are the sizes of the configuration (G groups of S tokens, widths M and H, E experts with
C positions per group; B sequences of length L, heads of width d).  Outputs, workspaces and packed gate
weights are made once in ``prepare``, as a server or a training loop keeps them.
"""
import numpy as np
import torch

import paper_2006_16668_amd as moe
from workloads import CONFIGS, MoEConfig, make_encoder_weights, make_inputs, make_upstream

DEV = "cuda:0"


def _layer(name, kind, cfg, prepacked=False):
    return {"name": name, "kind": kind, "G": cfg.G, "S": cfg.S, "M": cfg.M, "H": cfg.H, "E": cfg.E, "C": cfg.C,
            "dtype": cfg.act_dtype, "bias": cfg.logit_bias_std, "prepacked": prepacked}


def listed():
    shape = lambda G, S, M, H, E, C, dt="bf16": MoEConfig("", G=G, S=S, M=M, H=H, E=E, C=C, act_dtype=dt)
    return [
        # the smallest configuration of this repository, fp32: launches and latency only
        _layer("tiny_f32", "forward", CONFIGS["tiny"]),
        # a server's step: 64 tokens in flight through the paper-sized layer, whose expert weights
        # (1.07 GB) all have to be read for them
        _layer("serve_64_tokens", "forward", shape(1, 64, 1024, 8192, 32, 4), prepacked=True),
        # a batch of five sequences whose length is no multiple of anything
        _layer("odd_batch", "forward", shape(5, 700, 768, 3072, 24, 59), prepacked=True),
        # the paper-shaped share of one device: the headline workload of bench.py
        _layer("paper", "forward", CONFIGS["paper"], prepacked=True),
        # popular experts overflow, others leave their positions empty
        _layer("skewed", "forward", CONFIGS["skewed"], prepacked=True),
        # 17 GB of expert weights, the largest state
        _layer("many_experts", "forward", CONFIGS["many_experts"], prepacked=True),
        # training steps: the small configuration, an odd one, the paper's
        _layer("train_small", "train", CONFIGS["small"]),
        _layer("train_odd", "train", shape(3, 1333, 520, 2056, 12, 223)),
        _layer("train_paper", "train", CONFIGS["paper"]),
        # the precision the paper trained in, at a quarter of its width
        _layer("train_f32", "train", shape(4, 1024, 1024, 2048, 16, 128, "f32")),
        # self-attention over sequences that are not padded to a round length (paper's head sizes)
        {"name": "attention_1000", "kind": "attention", "B": 16, "L": 1000, "M": 1024, "heads": 16, "d": 128, "dtype": "bf16"},
        # a training step of the two encoder layers around the MoE layer, paper's attention sizes
        {"name": "encoder_train", "kind": "encoder", "B": 16, "L": 1024, "M": 1024, "H": 4096, "E": 2, "heads": 16, "d": 128, "dtype": "bf16"},
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "train", "train", "attention", "encoder"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    if kind in ("forward", "train"):
        E = _log(rng, 4, 128)
        G = rng.choice([1, 2, 3, 4, 6, 8])
        S = max(8, _log(rng, 64, 32768) // G)
        if rng.random() < 0.5:                       # widths of 256 and any multiple of 8
            M = 256 * rng.randint(1, 4)
            H = M * rng.choice([2, 4, 8])
        else:
            M = 8 * rng.randint(16, 128)
            H = 8 * (M * rng.choice([2, 3, 4]) // 8 + rng.randint(0, 9))
        while kind == "train" and E * M * H > 1 << 28 or 2 * G * S * M * H * (16 if dtype == "f32" else 1) > 1 << 39:
            H = 8 * (H // 16)                         # no more work than the paper's layer
        C = max(1, -(-2 * S // E))
        return {"kind": kind, "G": G, "S": S, "M": M, "H": H, "E": E, "C": C, "dtype": dtype,
                "bias": rng.choice([0.0, 0.0, 0.25]), "prepacked": kind == "forward" and rng.random() < 0.7}
    L = rng.choice([128 * rng.randint(1, 8), _log(rng, 16, 1000), _log(rng, 16, 1000)])
    d = rng.choice([64, 128])
    heads = rng.choice([4, 8, 16]) if d == 64 else rng.choice([2, 4, 8])
    B = max(1, _log(rng, 512, 8192 if dtype == "bf16" else 2048) // L)
    c = {"kind": kind, "B": B, "L": L, "M": 256 * rng.randint(1, 4), "heads": heads, "d": d, "dtype": dtype}
    if kind == "encoder":
        c.update(H=c["M"] * rng.choice([2, 4]), E=2)
    return c


def _config(case, seed):
    if case["kind"] in ("forward", "train"):
        return MoEConfig("case", G=case["G"], S=case["S"], M=case["M"], H=case["H"], E=case["E"], C=case["C"],
                         act_dtype=case["dtype"], seed=seed, logit_bias_std=case["bias"])
    # one group per sequence.  Two experts with room for every token: a token then meets the same
    # experts whichever of them comes first, so that rounding before the router (which no margin of
    # the inputs can keep from flipping a near tie) changes no output by more than rounding.
    return MoEConfig("case", G=case["B"], S=case["L"], M=case["M"], H=case.get("H", case["M"]), E=case.get("E", 2), C=case["L"],
                     act_dtype=case["dtype"], seed=seed)


def _bytes(n):
    return torch.empty(n, dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    cfg = _config(case, seed)
    sh = moe.MoEShape(cfg.G, cfg.S, cfg.M, cfg.H, cfg.E, cfg.C, cfg.act_dtype)
    kind = case["kind"]
    inp = make_inputs(cfg, device=DEV, condition=kind in ("forward", "train"), with_experts=kind != "attention")
    s = {"kind": kind, "sh": sh, "inp": inp, "y": torch.empty_like(inp.x),
         "aux": torch.empty(cfg.G, dtype=torch.float32, device=DEV)}
    if kind == "forward":
        s["ws"] = _bytes(moe.moe_workspace_bytes(sh))
        s["packed"] = None
        s["prepacked"] = case["prepacked"]
        if case["prepacked"]:
            n = moe.moe_gate_pack_bytes(sh)
            if n:
                s["packed"] = _bytes(n)
                moe.moe_gate_pack(sh, inp.wg, s["packed"])
    elif kind == "train":
        s["dy"], s["daux"] = make_upstream(cfg, device=DEV)
        s["fws"] = _bytes(moe.moe_train_workspace_bytes(sh))
        s["bws"] = _bytes(moe.moe_backward_workspace_bytes(sh))
        s["grads"] = [torch.empty_like(t) for t in (inp.x, inp.wg, inp.wi, inp.wo)]
    else:
        dims = s["dims"] = moe.EncoderDims(case["B"], case["L"], case["heads"], case["d"])
        w = make_encoder_weights(cfg, case["heads"], case["d"], device=DEV)
        if kind == "attention":
            s["wqkv"], s["wo_att"] = w["wqkv"][0], w["wo_att"][0]
            s["ws"] = _bytes(moe.moe_attention_workspace_bytes(sh, dims))
        else:
            inp.u.zero_()                            # the second expert always takes part
            s["weights"] = w = dict(w, wg=inp.wg, wi=inp.wi, wo=inp.wo)
            like = lambda v: [torch.empty_like(t) for t in v] if isinstance(v, list) else torch.empty_like(v)
            s["grads"] = {k: like(v) for k, v in w.items()}
            s["dx"] = torch.empty_like(inp.x)
            s["dy"], s["daux"] = make_upstream(cfg, device=DEV)
            s["fws"] = _bytes(moe.moe_encoder_train_workspace_bytes(sh, dims))
            s["bws"] = _bytes(moe.moe_encoder_backward_workspace_bytes(sh, dims))
    return s


def run(s):
    sh, i, y, aux = s["sh"], s["inp"], s["y"], s["aux"]
    if s["kind"] == "forward":
        if s["prepacked"]:
            moe.moe_forward_prepacked(sh, i.x, i.wg, s["packed"], i.u, i.wi, i.wo, y, aux, s["ws"])
        else:
            moe.moe_forward(sh, i.x, i.wg, i.u, i.wi, i.wo, y, aux, s["ws"])
        return y, aux
    if s["kind"] == "train":
        moe.moe_forward_train(sh, i.x, i.wg, i.u, i.wi, i.wo, y, aux, s["fws"])
        moe.moe_backward(sh, i.x, i.wg, i.wi, i.wo, s["dy"], s["daux"], s["fws"], *s["grads"], s["bws"])
        return y, aux, s["grads"]
    if s["kind"] == "attention":
        moe.moe_self_attention(sh, s["dims"], i.x, s["wqkv"], s["wo_att"], y, s["ws"])
        return y
    moe.moe_encoder_pair_forward_train(sh, s["dims"], i.x, s["weights"], i.u, y, aux, s["fws"])
    moe.moe_encoder_pair_backward(sh, s["dims"], i.x, s["weights"], s["dy"], s["daux"], s["fws"], s["dx"], s["grads"], s["bws"])
    return y, s["dx"], s["grads"]


def _routed(case):
    """(rows the experts multiply, experts with at least one row): one group simulated with logits of
    the inputs' distribution; which tokens they are does not matter for the amount of work."""
    G, S, E, C = case["G"], case["S"], case["E"], case["C"]
    rng = np.random.default_rng(1)
    z = rng.standard_normal((S, E), dtype=np.float32)
    if case["bias"]:
        z += case["bias"] * rng.standard_normal(E, dtype=np.float32)
    e1 = z.argmax(1)
    rows = np.arange(S)
    z1 = z[rows, e1].copy()
    z[rows, e1] = -np.inf
    e2 = z.argmax(1)
    sampled = 2 / (1 + np.exp(z1 - z[rows, e2])) > rng.random(S)
    kept = np.minimum(np.bincount(e1, minlength=E) + np.bincount(e2[sampled], minlength=E), C)
    total = G * int(kept.sum())
    return total, E if total >= 8 * E else int((kept > 0).sum())


def work(case):
    elt = 4 if case["dtype"] == "f32" else 2
    M = case["M"]
    if case["kind"] in ("forward", "train"):
        N, H, E = case["G"] * case["S"], case["H"], case["E"]
        rows, touched = _routed(case)
        experts, gate = 4 * rows * M * H, 2 * N * M * E
        weights = 2 * touched * M * H * elt
        data = N * M * elt
        if case["kind"] == "forward":
            return {"bytes": 2 * data + weights + M * E * 4 + N * 4, "flops": experts + gate}
        # x, dy in, y, dx out; weights in, their gradients out
        return {"bytes": 4 * data + weights + 2 * E * M * H * elt + 2 * M * E * 4 + N * 4, "flops": 3 * (experts + gate)}
    N, A = case["B"] * case["L"], case["heads"] * case["d"]
    att = 8 * N * M * A + 4 * N * case["L"] * A           # four projections, scores and context
    att_w = 4 * M * A * elt
    if case["kind"] == "attention":
        return {"bytes": 2 * N * M * elt + att_w, "flops": att}
    H, E = case["H"], case["E"]
    # backward: twice the forward's products, and the scores once more
    total = 3 * (2 * att + 4 * N * M * H * (1 + E)) + 2 * 2 * N * case["L"] * A
    return {"bytes": 4 * N * M * elt + 2 * (2 * att_w + 2 * (1 + E) * M * H * elt), "flops": total}


def tolerance(case):
    # measured against the same calls in fp32 (bf16) and in fp64 (fp32), about four times what was seen
    if case["kind"] in ("forward", "attention"):
        # bf16: operands, h and outputs rounded to 8 bits, 3e-3; fp32: sums over up to 8192 products, 9e-7
        return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 5e-6}
    # A gradient is also cut by relu' = [h > 0], and another order of the same sums moves some h across
    # 0: a share p of flipped elements shows as sqrt(p), alone in its place.
    if case["kind"] == "train":
        # bf16: 3e-3, 0.3 in a place; fp32: 2e-4 (a few of 16 million h), 0.1 in a place
        return {"rel": 1e-2, "max": 0.9} if case["dtype"] == "bf16" else {"rel": 8e-4, "max": 0.4}
    # encoder: what every h comes from is itself rounded on the way, 4e-3 of it in bf16 (5e-2 on the
    # gradients of wi, w1 then, 0.6 in a place), 3e-7 in fp32
    return {"rel": 3e-2, "max": 0.99} if case["dtype"] == "bf16" else {"rel": 1e-3, "max": 0.9}
