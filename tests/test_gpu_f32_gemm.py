"""The fp32 GEMM at the edges of its 64 and 128 tiles and 16-wide k steps, layers whose experts it packs
(M >= 128) and layers it does not: routing bit for bit, outputs and gradients against the oracle
within the tolerances of the randomly drawn shapes."""
import pytest

import test_gpu_random_shapes as shapes
from workloads import MoEConfig

pytestmark = pytest.mark.gpu


def _cfg(name, G, S, M, H, E, C, bias=0.0):
    return MoEConfig(name, G=G, S=S, M=M, H=H, E=E, C=C, act_dtype="f32", seed=9500 + G * C + M + H, logit_bias_std=bias)


CASES = [
    _cfg("one_row", 1, 40, 128, 4, 3, 1),
    _cfg("rows_63_k_tail_4", 1, 200, 132, 60, 3, 63),
    _cfg("rows_64", 2, 100, 144, 64, 4, 32),
    _cfg("rows_65_unpacked", 1, 150, 68, 124, 2, 65),
    _cfg("rows_129", 3, 140, 128, 132, 3, 43),
    _cfg("columns_252", 2, 90, 252, 260, 5, 40),
    _cfg("skewed", 4, 333, 192, 328, 9, 75, bias=1.0),
    # more row tiles than a band of eight: 64 x 128 and 64 x 64 tiles; 128 x 128 tiles, weight gradients in four groups
    _cfg("many_tiles", 2, 1400, 384, 520, 2, 700),
    _cfg("many_tiles_128", 2, 2600, 132, 132, 9, 577),
    # 128 x 128 tiles throughout
    _cfg("tiles_128", 2, 2100, 132, 132, 64, 65),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_forward_and_backward(cfg):
    shapes.test_random_shape(cfg)
