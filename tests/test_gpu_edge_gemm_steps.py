"""The tiled GEMM's forms with 64-wide k steps, two to four stages: sums that end inside a step, one row past
a tile, and each form in the forward products and the data gradients (256 compute units); and layers whose
products are formed by different kernels on either side of relu (persistent forward, tiled data gradient).
Routing bit for bit, outputs and gradients against the oracle within the tolerances of the drawn shapes."""
import pytest

import test_gpu_random_shapes as shapes
from workloads import MoEConfig

pytestmark = pytest.mark.gpu


def _cfg(name, G, S, M, H, E, C, bias=0.0):
    return MoEConfig(name, G=G, S=S, M=M, H=H, E=E, C=C, act_dtype="bf16", seed=9700 + G * C + M + H, logit_bias_std=bias)


CASES = [
    _cfg("64x64_deep_one_step", 1, 90, 128, 24, 2, 65),           # sums of 24 and of 128: less than a step, two steps
    _cfg("64x64_deep_tails", 2, 130, 136, 264, 2, 65),            # 128 + 8, 256 + 8
    _cfg("64x64", 1, 500, 136, 904, 12, 130),                     # 14 steps + 8
    _cfg("64x128", 2, 400, 168, 920, 24, 65),                     # 2 steps + 40, 14 + 24
    _cfg("64x128_deep", 2, 200, 184, 2056, 8, 65),                # 2 steps + 56
    _cfg("128x128", 3, 1000, 136, 2104, 12, 67, bias=0.5),
    _cfg("128x128_forward", 4, 2000, 136, 264, 12, 375),
    _cfg("128x128_deep", 1, 900, 520, 2056, 6, 200),
    _cfg("persistent_h_persistent_dh", 2, 1200, 256, 1536, 12, 256),
    _cfg("persistent_h_tiled_dh", 1, 2500, 256, 1024, 13, 515),
    _cfg("tiled_h_dh_without_bits", 2, 2500, 512, 2304, 20, 256),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_forward_and_backward(cfg):
    shapes.test_random_shape(cfg)
