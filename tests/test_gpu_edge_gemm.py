"""The tiled GEMM of shapes that are not made of whole 256-row tiles, at the edges of its tiles (64 x 64,
64 x 128, 128 x 128, 128 x 256, smaller ones for outputs of fewer tiles) and 32-wide k steps: routing bit for bit, outputs and gradients against the
oracle within the tolerances of the randomly drawn shapes.  G*C (rows per expert), M and H each take the
role of rows, columns and summed dimension over the six products of a step."""
import pytest

import test_gpu_random_shapes as shapes
from workloads import MoEConfig

pytestmark = pytest.mark.gpu


def _cfg(name, G, S, M, H, E, C, bias=0.0):
    return MoEConfig(name, G=G, S=S, M=M, H=H, E=E, C=C, act_dtype="bf16", seed=9000 + G * C + M + H, logit_bias_std=bias)


CASES = [
    # 64-row tiles (few of 64 columns, more of 128), their edges and k tails
    _cfg("rows_63", 1, 200, 136, 56, 3, 63),
    _cfg("rows_65_columns_72", 5, 60, 328, 72, 3, 13),
    _cfg("many_small_experts", 2, 300, 384, 1032, 100, 6),
    _cfg("one_row", 1, 40, 128, 8, 3, 1),
    _cfg("rows_127", 1, 300, 136, 120, 3, 127),
    _cfg("rows_128", 2, 150, 152, 128, 4, 64),
    _cfg("rows_129_k_tail_8", 3, 140, 136, 264, 3, 43),
    _cfg("rows_257", 1, 400, 264, 136, 2, 257),
    _cfg("columns_248", 5, 77, 248, 520, 4, 39),
    # enough tiles for the 128-row forms (h: 768 of 128 x 128; 512 of 128 x 256)
    _cfg("tiles_128x128", 2, 1500, 136, 904, 24, 195, bias=0.5),
    _cfg("tiles_128x256", 3, 1500, 144, 1000, 32, 130, bias=0.5),
    # more row tiles than a band of eight; nearly empty and overflowing experts
    _cfg("bands", 7, 400, 128, 256, 2, 171),
    _cfg("skewed", 4, 333, 192, 328, 9, 75, bias=1.0),
    # whole 256-row tiles, few of them: 128-row tiles for some products, the persistent kernel (whose
    # sums over k run to the next multiple of 256 rows) for others
    _cfg("few_tiles", 4, 300, 256, 2048, 12, 64),
    _cfg("few_tiles_skewed", 2, 512, 512, 1024, 16, 128, bias=1.0),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_forward_and_backward(cfg):
    shapes.test_random_shape(cfg)
