"""The persistent GEMM with row counts that are no multiple of its 256-row tiles: forward products with and
without recorded relu' bits, data gradients, packed rows and dense ones, the last expert's last tile (nothing is
read or written past an operand: the buffers here end where the operands end).  Large enough for the rule to take it
(256 compute units)."""
import pytest
import torch

import paper_2006_16668_amd as moe
import test_gpu_random_shapes as shapes
from workloads import MoEConfig

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# products the persistent kernel forms: all four; h and dh (with bits); out and dbuf; h and dh, a tile's last rows only;
# none (tiles of 64 x 128)
@pytest.mark.parametrize("G,S,M,H,E,C", [(1, 20500, 256, 256, 10, 4100), (1, 3700, 256, 2048, 8, 903), (2, 4100, 768, 256, 2, 4100),
                                         (1, 20400, 256, 768, 20, 2040), (2, 8200, 256, 256, 4, 4100)])
def test_forward_and_backward(G, S, M, H, E, C):
    shapes.test_random_shape(MoEConfig("rows", G=G, S=S, M=M, H=H, E=E, C=C, act_dtype="bf16", seed=9800 + C, logit_bias_std=0.0))


# persistent, persistent with one row in the last tile, tiles of 64 x 128
@pytest.mark.parametrize("rows,M,H", [(16000, 1024, 1024), (15873, 1024, 1024), (8209, 1024, 1024)])
def test_dense_rows(rows, M, H):
    g = torch.Generator(device=DEV).manual_seed(rows)
    u = torch.randn(rows, M, device=DEV, generator=g).bfloat16()
    w1 = (torch.randn(M, H, device=DEV, generator=g) / M ** 0.5).bfloat16()
    w2 = (torch.randn(H, M, device=DEV, generator=g) / H ** 0.5).bfloat16()
    # guard rows behind the results
    h = torch.full((rows + 300, H), 7.0, dtype=torch.bfloat16, device=DEV)
    out = torch.full((rows + 300, M), 7.0, dtype=torch.bfloat16, device=DEV)
    sh = moe.MoEShape(1, rows, M, H, 2, rows, "bf16")
    moe.moe_dense_ffn(sh, u.view(1, rows, M), w1, w2, h[:rows].view(1, rows, H), out[:rows].view(1, rows, M))
    torch.cuda.synchronize()
    want_h = torch.relu(u.float() @ w1.float())
    want = h[:rows].float() @ w2.float()
    # one bf16 rounding of the result: 2^-9 of it at most, 0.6 of that in the mean
    assert float((h[:rows].float() - want_h).norm() / want_h.norm()) < 2.0 ** -8.5
    assert float((out[:rows].float() - want).norm() / want.norm()) < 2.0 ** -8.5
    assert bool((h[rows:] == 7).all()) and bool((out[rows:] == 7).all())
