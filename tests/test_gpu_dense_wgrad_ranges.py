"""Weight gradients of the dense encoder layers summed over ranges of tokens: token counts that no range
length divides, ranges shorter than a k step left over, one range only; all gradients of the pair against the
oracle within the tolerances of test_gpu_encoder_backward."""
import pytest

import test_gpu_encoder_backward as enc
from workloads import MoEConfig

pytestmark = pytest.mark.gpu


def _cfg(G, S, M, H):
    return MoEConfig("ranges", G=G, S=S, M=M, H=H, E=2, C=S, act_dtype="bf16", seed=9900 + G * S + M, logit_bias_std=0.0)


# tokens: 130 (one range), 1030 (ranges of 160 or 128, 6 left), 1536 (even), 1201 (odd)
@pytest.mark.parametrize("B,L,M,H,heads,d", [(1, 130, 128, 136, 2, 64), (5, 206, 136, 264, 2, 64), (3, 512, 256, 512, 4, 64),
                                             (1, 1201, 104, 256, 1, 128)])
def test_encoder_pair_backward(B, L, M, H, heads, d):
    enc.test_encoder_pair_backward(_cfg(B, L, M, H), B, L, heads, d)
