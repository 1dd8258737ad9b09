"""Sequence lengths that are no multiple of the attention kernels' 128-row blocks: forward and all
gradients of the encoder pair against the oracle, with the stage-wise checks and tolerances of the
fixed cases.  Lengths around the edges of the 32-row wavefront tiles, the 64-row staged blocks and
the 128-row workgroups, one of several blocks, for both head sizes."""
import numpy as np
import pytest
import torch

import paper_2006_16668_amd as moe
import test_gpu_encoder_backward as pair
from harness import f64, rel_fro, shape_of
from oracle import transformer_oracle as tro
from test_gpu_encoder import _split_qkv
from workloads import MoEConfig, make_encoder_weights, make_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _cfg(B, L, seed):
    return MoEConfig(f"L{L}", G=B, S=L, M=128, H=64, E=4, C=max(1, L // 2), act_dtype="bf16", seed=seed)


@pytest.mark.parametrize("L,d", [(33, 64), (63, 128), (65, 128), (127, 64), (129, 64), (200, 128), (333, 64)])
def test_pair_forward_and_backward(L, d):
    B = max(2, 256 // L)
    pair.test_encoder_pair_backward(_cfg(B, L, 600 + L), B, L, 2, d)


@pytest.mark.parametrize("L,d", [(1, 64), (2, 128), (31, 128), (64, 64), (96, 128), (128, 64), (384, 128), (1000, 128)])
def test_self_attention(L, d):
    B, heads = 3, 3
    cfg = _cfg(B, L, 700 + L)
    dims = moe.EncoderDims(B, L, heads, d)
    sh = shape_of(cfg)
    inp = make_inputs(cfg, device=DEV, condition=False)
    w = make_encoder_weights(cfg, heads, d, device=DEV)
    # sharper scores than random projections give, so that a wrongly masked key cannot hide
    wqkv = w["wqkv"][0].clone()
    wqkv[:, :2 * heads * d] *= 2
    ws = torch.empty(moe.moe_attention_workspace_bytes(sh, dims), dtype=torch.uint8, device=DEV)
    out = torch.full_like(inp.x, float("nan"))
    moe.moe_self_attention(sh, dims, inp.x, wqkv, w["wo_att"][0], out, ws)
    torch.cuda.synchronize()
    want = tro.self_attention(f64(inp.x), *_split_qkv(wqkv, heads * d), f64(w["wo_att"][0]), heads)
    # q, k, v, p and ctx are rounded to 8 bits once each: a few 2^-9 (scores up to about 4: their
    # rounding enters the exponent, 4 * 2^-9)
    assert rel_fro(f64(out), want) < 2e-2
    rows = np.linalg.norm(f64(out) - want, axis=-1) / np.linalg.norm(want, axis=-1)
    assert rows.max() < 6e-2, rows.max()


@pytest.mark.parametrize("L,d", [(130, 64), (200, 128), (257, 128), (257, 64), (321, 128), (900, 64), (384, 128)])
def test_self_attention_with_a_full_chip(L, d):
    """Three and more key blocks with at least two workgroups on every compute unit, most lengths with
    wavefronts that hold no query and so run ahead of the others: a stage must not be refilled before
    all of them have read it.  Every row against the oracle, and the same bits on a second call."""
    heads = 16
    B = -(-512 // (heads * -(-L // 128)))
    print(f"L={L} d={d} B={B}", flush=True)
    cfg = _cfg(B, L, 800 + L)
    dims = moe.EncoderDims(B, L, heads, d)
    sh = shape_of(cfg)
    inp = make_inputs(cfg, device=DEV, condition=False)
    w = make_encoder_weights(cfg, heads, d, device=DEV)
    wqkv = w["wqkv"][0].clone()
    wqkv[:, :2 * heads * d] *= 2
    ws = torch.empty(moe.moe_attention_workspace_bytes(sh, dims), dtype=torch.uint8, device=DEV)
    outs = [torch.full_like(inp.x, float("nan")) for _ in range(2)]
    for out in outs:
        moe.moe_self_attention(sh, dims, inp.x, wqkv, w["wo_att"][0], out, ws)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])
    want = tro.self_attention(f64(inp.x), *_split_qkv(wqkv, heads * d), f64(w["wo_att"][0]), heads)
    got = f64(outs[0])
    assert rel_fro(got, want) < 2e-2                      # as above
    rows = np.linalg.norm(got - want, axis=-1) / np.linalg.norm(want, axis=-1)
    assert rows.max() < 6e-2, rows.max()


@pytest.mark.parametrize("L,d,block", [(200, 64, 0), (200, 128, 64), (333, 128, 128), (256, 64, 0)])
def test_a_block_of_keys_with_scores_of_minus_infinity(L, d, block):
    """64 consecutive keys, the first ones among them, whose finite products overflow to -inf: they get
    probability 0, whichever block they are in."""
    M = max(3 * d, -(-L // 8) * 8)
    cfg = MoEConfig("inf", G=1, S=L, M=M, H=64, E=2, C=L, act_dtype="bf16", seed=5)
    dims, sh = moe.EncoderDims(1, L, 1, d), shape_of(cfg)
    gen = torch.Generator(device=DEV).manual_seed(L + d)
    x = torch.zeros((1, L, M), device=DEV, dtype=torch.bfloat16)
    x[0, torch.arange(L), torch.arange(L)] = 1            # token t: q, k, v are row t of wqkv
    w = torch.randn((M, 3 * d), generator=gen, device=DEV)
    w[:, 0], w[:, d] = 2.0 ** 70, w[:, d] * 2.0 ** -70
    w[block:block + 64, d] = -2.0 ** 70
    wqkv = w.to(torch.bfloat16)
    eye = torch.zeros((d, M), device=DEV, dtype=torch.bfloat16)
    eye[torch.arange(d), torch.arange(d)] = 1
    out = torch.full_like(x, float("nan"))
    moe.moe_self_attention(sh, dims, x, wqkv, eye, out,
                           torch.empty(moe.moe_attention_workspace_bytes(sh, dims), dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    want = tro.self_attention(f64(x), *_split_qkv(wqkv, d), f64(eye), 1)
    rows = np.linalg.norm(f64(out) - want, axis=-1) / np.linalg.norm(want, axis=-1)
    assert rows.max() < 1e-2, rows.max()                  # probabilities and ctx rounded to 8 bits
