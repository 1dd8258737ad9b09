"""The fp32 attention core on the matrix cores: lengths at the edges of its blocks of 32, wavefronts with columns of
their own and sharing them, against float64; scores that overflow to -inf; its backward pass through the encoder
pair.  The projections pass q, k, v and the context through unchanged (identity weights)."""
import pytest
import torch

import paper_2006_16668_amd as moe
import test_gpu_encoder_backward as enc
from workloads import MoEConfig

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _attention(q, k, v):
    B, L, heads, d = q.shape
    A = heads * d
    u = torch.cat([t.reshape(B, L, A) for t in (q, k, v)], dim=-1).contiguous()
    out = torch.full_like(u, float("nan"))
    sh, dims = moe.MoEShape(B, L, 3 * A, 8, 2, L, "f32"), moe.EncoderDims(B, L, heads, d)
    ws = torch.empty(moe.moe_attention_workspace_bytes(sh, dims), dtype=torch.uint8, device=DEV)
    wo = torch.eye(A, 3 * A, device=DEV)
    moe.moe_self_attention(sh, dims, u, torch.eye(3 * A, device=DEV), wo, out, ws)
    torch.cuda.synchronize()
    return out[..., :A].reshape(B, L, heads, d)


def _want(q, k, v):
    s = torch.einsum("blhd,bmhd->bhlm", q.double().cpu(), k.double().cpu()) / q.shape[-1] ** 0.5
    return torch.einsum("bhlm,bmhd->blhd", torch.softmax(s, dim=-1), v.double().cpu())


# 2 x 64 columns of blocks and fewer share columns unless a sequence is one block; 40 x 33 x 16 has columns for all
@pytest.mark.parametrize("B,L,heads,d", [(64, 1, 2, 64), (5, 31, 1, 128), (4, 32, 2, 64), (4, 33, 1, 64), (1, 129, 2, 128),
                                         (2, 257, 2, 64), (1, 160, 1, 128), (40, 33, 16, 64), (34, 95, 4, 128)])
def test_against_float64(B, L, heads, d):
    g = torch.Generator(device=DEV).manual_seed(B + L + d)
    q, k, v = (torch.randn(B, L, heads, d, device=DEV, generator=g) for _ in range(3))
    got, want = _attention(q, k, v).cpu().double(), _want(q, k, v)
    # a score of |s| < 8 carries 2^-24 (sqrt(d) / 2 + |s|) at most, p and the sums a few 2^-24 more
    assert float((got - want).norm() / want.norm()) < 1e-6


@pytest.mark.parametrize("B,L,heads,d", [(1, 200, 2, 64), (40, 70, 16, 64)])
def test_scores_of_minus_infinity_add_nothing(B, L, heads, d):
    g = torch.Generator(device=DEV).manual_seed(L)
    q, k, v = (torch.randn(B, L, heads, d, device=DEV, generator=g) for _ in range(3))
    q[..., 0] = 1e15
    k[..., 0] = 0
    k[:, :40, :, 0] = -1e25                                    # the whole first block of keys and part of the second
    got = _attention(q, k, v).cpu().double()
    q[..., 0] = 0
    want = _want(q, k[:, 40:], v[:, 40:])
    assert float((got - want).norm() / want.norm()) < 1e-6


# columns of their own: 3 x 33, 36 x 40, 3 x 40 and 2 x 31; shared: 2 x 95, 1 x 257, and 1 x 170 (two blocks of rows to a
# wavefront at d = 128)
@pytest.mark.parametrize("B,L,heads,d", [(3, 33, 2, 64), (2, 95, 1, 128), (1, 257, 2, 64), (36, 40, 16, 64), (3, 40, 2, 128),
                                         (2, 31, 3, 128), (1, 170, 2, 128)])
def test_backward(B, L, heads, d):
    enc.test_encoder_pair_backward(MoEConfig("f32", G=B, S=L, M=64, H=72, E=2, C=L, act_dtype="f32", seed=9600 + L,
                                             logit_bias_std=0.0), B, L, heads, d)


@pytest.mark.parametrize("B,L,heads,d,last", [(2, 200, 2, 64, True), (40, 70, 16, 64, True), (1, 97, 2, 128, True), (34, 95, 4, 128, True),
                                              (1, 96, 2, 64, True), (2, 200, 2, 64, False)])
def test_infinite_value(B, L, heads, d, last):
    """One infinite element of v makes its column of the context infinite, wherever its row stands: blocks of 32 rows
    are filled up with others than copies of it."""
    g = torch.Generator(device=DEV).manual_seed(L + d)
    A = heads * d
    u = torch.randn(B, L, 3 * A, device=DEV, generator=g)
    w = torch.eye(3 * A, device=DEV)
    col = 2 * A + 5                                            # element 5 of v of the first head
    w[col, col] = 2
    u[:, L - 1 if last else 3, col] = 3e38
    out = torch.zeros_like(u)
    sh, dims = moe.MoEShape(B, L, 3 * A, 8, 2, L, "f32"), moe.EncoderDims(B, L, heads, d)
    ws = torch.empty(moe.moe_attention_workspace_bytes(sh, dims), dtype=torch.uint8, device=DEV)
    moe.moe_self_attention(sh, dims, u, w, torch.eye(A, 3 * A, device=DEV), out, ws)
    torch.cuda.synchronize()
    assert bool((out[..., 5] == float("inf")).all())
