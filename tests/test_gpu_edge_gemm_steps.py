"""The tiled GEMM's forms with 64-wide k steps, two to four stages: sums that end inside a step, one row past
a tile, and each form in the forward products and the data gradients (256 compute units); and layers whose
h and dh are both formed by the persistent kernel, also where inference takes a tiled form for h (same bits).
Routing bit for bit, outputs and gradients against the oracle within the tolerances of the drawn shapes."""
import pytest
import torch

import test_gpu_random_shapes as shapes
from harness import gpu_forward, gpu_forward_backward
from workloads import MoEConfig, make_inputs, make_upstream

pytestmark = pytest.mark.gpu


def _cfg(name, G, S, M, H, E, C, bias=0.0):
    return MoEConfig(name, G=G, S=S, M=M, H=H, E=E, C=C, act_dtype="bf16", seed=9700 + G * C + M + H, logit_bias_std=bias)


CASES = [
    _cfg("64x64_deep_one_step", 1, 90, 128, 24, 2, 65),           # sums of 24 and of 128: less than a step, two steps
    _cfg("64x64_deep_tails", 2, 130, 136, 264, 2, 65),            # 128 + 8, 256 + 8
    _cfg("64x64", 1, 500, 136, 904, 12, 130),                     # dh; h 64x128_deep; 14 steps + 8
    _cfg("64x64_forward", 1, 300, 264, 2056, 8, 65),              # 4 steps + 8
    _cfg("64x128", 2, 400, 168, 920, 24, 65),                     # 2 steps + 40, 14 + 24
    _cfg("64x128_deep", 2, 200, 184, 2056, 8, 65),                # 2 steps + 56
    _cfg("128x128", 3, 1000, 136, 2104, 12, 67, bias=0.5),
    _cfg("64x64_and_64x128_many_rows", 4, 2000, 136, 264, 12, 375),
    _cfg("128x128_deep", 1, 900, 520, 2056, 6, 200),
    _cfg("64x128_whole_row_tiles", 2, 1200, 256, 1536, 12, 256),
    _cfg("64x128_deep_h_64x128_dh", 1, 2500, 256, 1024, 13, 515),
    _cfg("128x256_h_128x128_dh", 2, 2500, 512, 2304, 20, 256),
    _cfg("persistent_h_dh", 1, 2200, 128, 2304, 3, 1536),
    _cfg("persistent_h_dh_rows", 1, 2200, 128, 2304, 8, 515),
    _cfg("persistent_h_dh_in_training", 1, 15400, 256, 1536, 20, 1536),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_forward_and_backward(cfg):
    shapes.test_random_shape(cfg)


def test_training_and_inference_take_different_forms_of_h():
    cfg = CASES[-1]
    inp = make_inputs(cfg, device="cuda:0")
    y, _ = gpu_forward(cfg, inp)
    dy, daux = make_upstream(cfg, device="cuda:0")
    assert torch.equal(gpu_forward_backward(cfg, inp, dy, daux)["y"], y)
