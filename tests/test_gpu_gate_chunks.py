"""The one-chunk-per-block gate kernel at the edges of its ranges (fp32: E <= 128, bf16: E <= 64): feature
counts around its 32 / 64-feature blocks and their split over the wavefronts, expert counts around
the 32-expert tiles, one token to several ragged chunks, and a single chunk in all (which skips the
scan and the slots kernel), against the oracle: integers bit for bit, floats to 1e-5."""
import pytest

import test_gpu_random_shapes as shapes
from harness import assert_gate_floats_close, assert_routing_equal, gpu_gate
from oracle import moe_oracle as orc
from workloads import MoEConfig, make_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("G,S,M,E,C,dt", [
    (1, 1, 4, 2, 1, "f32"), (1, 63, 36, 3, 11, "f32"), (1, 64, 256, 128, 1, "f32"), (2, 64, 260, 33, 4, "f32"),
    (3, 65, 1024, 65, 2, "f32"), (1, 200, 2052, 100, 3, "f32"), (2, 129, 96, 64, 5, "f32"), (4, 256, 128, 31, 20, "f32"),
    (1, 1, 8, 2, 1, "bf16"), (1, 64, 1024, 32, 4, "bf16"), (1, 50, 520, 33, 1, "bf16"), (5, 63, 64, 64, 2, "bf16"),
    (2, 300, 1032, 7, 90, "bf16"), (3, 128, 456, 40, 7, "bf16")])
def test_gate(G, S, M, E, C, dt):
    cfg = MoEConfig("gate", G=G, S=S, M=M, H=8, E=E, C=C, act_dtype=dt, seed=800 + S + M + E)
    inp = make_inputs(cfg, device=DEV)
    x, wg, u = inp.host_f64()
    gates = orc.softmax_gates(x, wg)
    want = orc.top2_gating(gates, u, C)
    r = gpu_gate(cfg, inp.x, inp.wg, inp.u)
    assert_routing_equal(r, want)
    assert_gate_floats_close(r, want, gates=gates)


@pytest.mark.parametrize("S,E,C", [(1, 2, 1), (37, 5, 9), (64, 32, 4), (64, 3, 64)])
def test_layer_of_a_single_chunk_packs_its_rows(S, E, C):
    shapes.test_random_shape(MoEConfig("chunk", G=1, S=S, M=136, H=72, E=E, C=C, act_dtype="bf16", seed=850 + S + E))
