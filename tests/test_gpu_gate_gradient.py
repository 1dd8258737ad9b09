"""The gate's gradient kernels at the edges of their ranges: token counts around the 32-token stages and
64-token tiles, widths around the 128-feature tiles, expert counts around the 32-expert tiles and their
groups of four (and one expert more than the bf16 GEMM form starts at), both element types; all
gradients against the oracle within the tolerances of the randomly drawn shapes."""
import pytest

import test_gpu_random_shapes as shapes
from workloads import MoEConfig

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,S,M,E,dt", [
    (1, 31, 8, 2, "bf16"), (1, 33, 120, 16, "f32"), (3, 43, 136, 17, "bf16"), (1, 64, 128, 32, "f32"),
    (2, 65, 264, 33, "bf16"), (1, 127, 132, 64, "f32"), (4, 200, 520, 65, "bf16"), (2, 129, 72, 100, "f32"),
    (1, 300, 256, 128, "bf16"), (3, 111, 124, 129, "f32"), (2, 128, 256, 130, "bf16")])
def test_backward(G, S, M, E, dt):
    shapes.test_random_shape(MoEConfig("dz", G=G, S=S, M=M, H=24, E=E, C=max(2, 3 * S // E), act_dtype=dt,
                                       seed=8800 + S + M + E))
