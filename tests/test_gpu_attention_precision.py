"""bf16 attention over sequences that are no multiple of 128 long: probabilities and their gradients stay
fp32 until they have been multiplied.

The calls are set up so that q, k, v and the upstream gradient are known exactly (selections by one-hot rows,
weights of the other sub-layers zero) and the core's results come out unchanged but for their own rounding
to bf16.  What is left is compared with float64: half a bf16 unit in the last place of the result plus
2^-18 of the sum of the products' magnitudes.  Derivation: fp32 scores, exponent arguments (up to 2^4),
row statistic and gradients of scores carry a few 2^-24 each, relative to magnitudes that the bound contains:
some 2^-20 in all.  A probability rounded to bf16 is off by up to 2^-9."""
import numpy as np
import pytest
import torch

import paper_2006_16668_amd as moe
from harness import f64
from workloads import MoEConfig, make_encoder_weights

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
RAGGED = [(200, 64), (200, 128), (65, 128), (333, 64), (130, 64), (321, 128)]


def excess(got, want, magnitude):
    """Largest error beyond the result's own rounding, relative to the magnitude of its sum."""
    half_ulp = np.exp2(np.floor(np.log2(np.maximum(np.abs(want), 1e-300))) - 8)
    return float(((np.abs(got - want) - half_ulp).clip(0) / magnitude).max())


def core(L, d, heads, seed):
    """Forward and backward of the core for one sequence: (q, k, v, dctx), ctx and dq, dk, dv as float64
    [heads, L, d] arrays of the bf16 values."""
    A, M = heads * d, max(heads * d, -(-L // 8) * 8)
    cfg = MoEConfig("exact", G=1, S=L, M=M, H=64, E=2, C=L, act_dtype="bf16", seed=seed)
    sh = moe.MoEShape(1, L, M, 64, 2, L, "bf16")
    dims = moe.EncoderDims(1, L, heads, d)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rnd = lambda *s: torch.randn(s, generator=gen, device=DEV)
    new = lambda n: torch.empty(n, dtype=torch.uint8, device=DEV)
    w = make_encoder_weights(cfg, heads, d, device=DEV)
    for name in ("w1", "w2"):
        w[name].zero_()
    w["wqkv"][1].zero_()
    w["wo_att"][1].zero_()
    # token t is the one-hot row t after layer normalisation, its q, k, v are row t of wqkv
    x = torch.zeros((1, L, M), device=DEV, dtype=torch.bfloat16)
    x[0, torch.arange(L), torch.arange(L)] = 1.0
    sd = float(np.sqrt((1 / M) * (1 - 1 / M) + 1e-6))
    w["ln_gamma"][0].fill_(sd)
    w["ln_beta"][0].fill_(1 / M)
    n1 = torch.empty_like(x)
    moe.moe_add_layer_norm(sh, x, None, w["ln_gamma"][0], w["ln_beta"][0], None, n1)
    assert (n1[x == 1] == 1).all() and (n1[x == 0].abs().max() < 1e-6)
    qkv = rnd(M, 3 * A)
    qkv[:, :A] *= 1.5
    w["wqkv"][0] = qkv.to(torch.bfloat16)
    eye = torch.zeros((A, M), device=DEV, dtype=torch.bfloat16)
    eye[torch.arange(A), torch.arange(A)] = 1.0
    w["wo_att"][0] = eye
    onehot = x.clone()                                   # ctx as the training forward stores it
    ctx = torch.empty_like(x)
    moe.moe_self_attention(sh, dims, onehot, w["wqkv"][0], eye, ctx, new(moe.moe_attention_workspace_bytes(sh, dims)))
    wi = torch.zeros((2, M, 64), device=DEV, dtype=torch.bfloat16)
    wo = torch.zeros((2, 64, M), device=DEV, dtype=torch.bfloat16)
    weights = dict(w, wg=torch.zeros((M, 2), device=DEV), wi=wi, wo=wo)
    dy, daux = rnd(1, L, M).to(torch.bfloat16), torch.zeros(1, device=DEV)
    y, aux, dx = torch.empty_like(x), torch.empty(1, device=DEV), torch.empty_like(x)
    like = lambda v: [torch.empty_like(t) for t in v] if isinstance(v, list) else torch.empty_like(v)
    grads = {k: like(v) for k, v in weights.items()}
    fws, bws = new(moe.moe_encoder_train_workspace_bytes(sh, dims)), new(moe.moe_encoder_backward_workspace_bytes(sh, dims))
    u = torch.full((1, L), 0.5, device=DEV)
    moe.moe_encoder_pair_forward_train(sh, dims, x, weights, u, y, aux, fws)
    moe.moe_encoder_pair_backward(sh, dims, x, weights, dy, daux, fws, dx, grads, bws)
    torch.cuda.synchronize()
    split = lambda t: [f64(t)[:L, i * A:(i + 1) * A].reshape(L, heads, d).transpose(1, 0, 2) for i in range(t.shape[-1] // A)]
    return (*split(w["wqkv"][0]), split(dy[0, :, :A])[0]), split(ctx[0, :, :A])[0], split(grads["wqkv"][0])


def errors(L, d, heads, seed):
    (q, k, v, g), ctx, (dq, dk, dv) = core(L, d, heads, seed)
    T = lambda a: a.transpose(0, 2, 1)
    s = q @ T(k) / np.sqrt(d)
    p = np.exp(s - s.max(-1, keepdims=True))
    p /= p.sum(-1, keepdims=True)
    dp, dvec = g @ T(v), (g * ctx).sum(-1, keepdims=True)
    ds = p * (dp - dvec) / np.sqrt(d)
    mag = p * (np.abs(g) @ T(np.abs(v)) + (np.abs(g) * np.abs(ctx)).sum(-1, keepdims=True)) / np.sqrt(d)
    return {"ctx": excess(ctx, p @ v, p @ np.abs(v)), "dq": excess(dq, ds @ k, mag @ np.abs(k)),
            "dk": excess(dk, T(ds) @ q, T(mag) @ np.abs(q)), "dv": excess(dv, T(p) @ g, T(p) @ np.abs(g))}


@pytest.mark.parametrize("L,d", RAGGED)
def test_products_of_fp32_probabilities(L, d):
    err = errors(L, d, 2, 1000 + L + d)
    print(f"L={L} d={d}", {k: f"{v:.1e}" for k, v in err.items()}, flush=True)
    for name, e in err.items():
        assert e < 2.0 ** -18, (name, e)
