"""The one-chunk-per-block gate kernel at the edges of its ranges (fp32: E <= 128, bf16: E <= 64): feature
counts around its 32 / 64-feature blocks and their split over the wavefronts, expert counts around
the 32-expert tiles, one token to several ragged chunks, and a single chunk in all (which skips the
scan and the slots kernel), against the oracle: integers bit for bit, floats to 1e-5.  Likewise the kernel
that counts positions in one launch, around its 512 chunks, its 16 384 counters and its expert widths, and
the two kernels past them."""
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


ROUTE = [  # G, S, M, E, C: one launch up to 512 chunks, 128 experts, 16384 counters; two past that
    (512, 1, 16, 5, 1), (513, 1, 16, 5, 1), (128, 2, 64, 128, 1), (129, 2, 64, 128, 1), (7, 70, 64, 129, 2),
    (3, 1100, 32, 16, 150), (2, 2200, 32, 17, 200), (1, 4200, 32, 33, 260), (9, 130, 64, 65, 3), (70, 65, 16, 2, 40)]


@pytest.mark.parametrize("G,S,M,E,C", ROUTE)
def test_positions(G, S, M, E, C):
    test_gate(G, S, M, E, C, "bf16")


@pytest.mark.parametrize("G,S,E,C", [(512, 1, 5, 1), (513, 1, 5, 1), (37, 3, 17, 1), (3, 1100, 16, 150), (18, 66, 65, 2)])
def test_row_maps(G, S, E, C):
    shapes.test_random_shape(MoEConfig("route", G=G, S=S, M=136, H=72, E=E, C=C, act_dtype="bf16", seed=870 + S + E))


@pytest.mark.parametrize("S,E,C", [(1, 2, 1), (37, 5, 9), (64, 32, 4), (64, 3, 64)])
def test_layer_of_a_single_chunk_packs_its_rows(S, E, C):
    shapes.test_random_shape(MoEConfig("chunk", G=1, S=S, M=136, H=72, E=E, C=C, act_dtype="bf16", seed=850 + S + E))


@pytest.mark.parametrize("G,S,E,C", [
    # counted in one launch: groups of one, two and three chunks, eight or one of them summed at a time
    (100, 5, 6, 2), (60, 70, 20, 8), (9, 128, 100, 3), (40, 150, 3, 60),
    # sums by a launch of its own from 17 groups on, around its 32 segments and their batches of eight
    (16, 2060, 5, 500), (17, 1990, 5, 500), (31, 3, 130, 1), (33, 3, 130, 1), (257, 2, 140, 1), (600, 3, 9, 1), (1030, 2, 4, 1)])
def test_row_maps_of_many_groups(G, S, E, C):
    shapes.test_random_shape(MoEConfig("groups", G=G, S=S, M=136, H=72, E=E, C=C, act_dtype="bf16", seed=880 + G + S + E))
