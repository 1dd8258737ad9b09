"""bf16 attention: a sequence's context and gradients do not depend on how many other sequences come with it.

Few and many (sequence, head) pairs take different kernels: dk and dv of 64 keys per wavefront where d is 128 and the
blocks of 128 keys fill the device more than once; of ragged lengths, the short dq kernel for few of them up to 255 tokens of
d 128 and for many from 256 of d 64 on.  The sums run in one order in all of them, so the results are compared bit for
bit.  Lengths: one block of 64 rows, its edges, 128 and 256 columns and their edges, several.  At most 16384 tokens:
gates of more take another order of sums."""
import pytest
import torch

import paper_2006_16668_amd as moe
from workloads import MoEConfig, make_encoder_weights, make_inputs, make_upstream

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def step(B, L, heads, d, x, dy, w, u):
    sh = moe.MoEShape(B, L, 256, 256, 2, L, "bf16")
    dims = moe.EncoderDims(B, L, heads, d)
    new = lambda n: torch.empty(n, dtype=torch.uint8, device=DEV)
    y, aux = torch.empty_like(x), torch.empty(B, device=DEV)
    fws = new(moe.moe_encoder_train_workspace_bytes(sh, dims))
    moe.moe_encoder_pair_forward_train(sh, dims, x, w, u, y, aux, fws)
    like = lambda v: [torch.empty_like(t) for t in v] if isinstance(v, list) else torch.empty_like(v)
    grads, dx = {k: like(v) for k, v in w.items()}, torch.empty_like(x)
    moe.moe_encoder_pair_backward(sh, dims, x, w, dy, torch.zeros(B, device=DEV), fws, dx, grads,
                                  new(moe.moe_encoder_backward_workspace_bytes(sh, dims)))
    return y, dx


# two of each are the few.  WIDE: the many take the dk, dv kernel of 64 keys per wavefront (L 384 and 640: its last block has
# wavefronts without keys, which only stage)
WIDE = [(128, 8, 256, 40), (128, 8, 512, 24), (128, 8, 384, 16), (128, 8, 640, 8)]
OTHERS = [(128, 8, 384, 40), (64, 8, 256, 40), (64, 8, 128, 70), (128, 8, 129, 24), (128, 8, 200, 40), (128, 8, 321, 24),
          (64, 8, 257, 24), (64, 8, 449, 24)]


@pytest.mark.parametrize("d,heads,L,B", WIDE + OTHERS)
def test_many_sequences_give_the_bits_of_few(d, heads, L, B):
    cfg = MoEConfig("blocks", G=B, S=L, M=256, H=256, E=2, C=L, act_dtype="bf16", seed=5)
    inp = make_inputs(cfg, device=DEV, condition=False, with_experts=True)
    dy, _ = make_upstream(cfg, device=DEV)
    w = dict(make_encoder_weights(cfg, heads, d, device=DEV), wg=inp.wg, wi=inp.wi, wo=inp.wo)
    inp.u.zero_()
    y, dx = step(B, L, heads, d, inp.x, dy, w, inp.u)
    for first in (0, B - 2):                            # two sequences alone, from both ends
        part = slice(first, first + 2)
        y2, dx2 = step(2, L, heads, d, inp.x[part].contiguous(), dy[part].contiguous(), w, inp.u[part].clone())
        assert torch.equal(y[part], y2)
        assert torch.equal(dx[part], dx2)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L", [1, 17, 31, 32, 33, 48, 49, 63, 64, 65, 127, 128, 129, 191, 255, 256, 257, 384, 449, 640])
def test_core_against_float64_at_the_edges_of_blocks(L, d):
    """ctx through moe_self_attention with an identity output projection.  q, k, v are rounded to bf16 by their own
    projection, which the reference takes from the same product in float64 and rounds: half a unit in the last place of
    either (2^-9 each) moves a score of magnitude ~1 by 2^-8, ctx (a mean of values ~1) by at most 2^-7 of the row's
    norm with its own rounding and that of P (2^-9): 1e-2 with room for none of them aligning."""
    heads, B, M = 2, 2, 2 * d
    A = heads * d
    sh = moe.MoEShape(B, L, M, 64, 2, L, "bf16")
    dims = moe.EncoderDims(B, L, heads, d)
    gen = torch.Generator(device=DEV).manual_seed(L * 131 + d)
    x = torch.randn((B, L, M), generator=gen, device=DEV).to(torch.bfloat16)
    wqkv = (torch.randn((M, 3 * A), generator=gen, device=DEV) / M ** 0.5).to(torch.bfloat16)
    eye = torch.eye(A, device=DEV).to(torch.bfloat16)
    out = torch.empty_like(x)
    moe.moe_self_attention(sh, dims, x, wqkv, eye, out, torch.empty(moe.moe_attention_workspace_bytes(sh, dims), dtype=torch.uint8, device=DEV))
    qkv = (x.cpu().double() @ wqkv.cpu().double()).to(torch.bfloat16).double().view(B, L, 3, heads, d)
    q, k, v = (qkv[:, :, i].transpose(1, 2).contiguous() for i in range(3))
    p = torch.softmax(q @ k.transpose(-1, -2).contiguous() / d ** 0.5, -1)
    want = (p @ v).transpose(1, 2).reshape(B, L, A)
    got = out.cpu().double()
    assert torch.isfinite(got).all()
    err = (got - want).norm(dim=-1) / want.norm(dim=-1)
    assert err.max() < 1e-2, (L, d, float(err.max()), int(err.argmax()))
