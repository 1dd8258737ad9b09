"""The gate's gradient kernels at the edges of their ranges: token counts around the 32-token stages and
64-token tiles, widths around the 128-feature tiles, expert counts around the 32-expert tiles and their
groups of four (and one expert more than the bf16 GEMM form starts at), both element types; all
gradients against the oracle within the tolerances of the randomly drawn shapes."""
import pytest
import torch

import paper_2006_16668_amd as moe
import test_gpu_random_shapes as shapes
from harness import gpu_forward_backward, shape_of
from workloads import MoEConfig, make_inputs, make_upstream

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("G,S,M,E,dt", [
    (1, 31, 8, 2, "bf16"), (1, 33, 120, 16, "f32"), (3, 43, 136, 17, "bf16"), (1, 64, 128, 32, "f32"),
    (2, 65, 264, 33, "bf16"), (1, 127, 132, 64, "f32"), (4, 200, 520, 65, "bf16"), (2, 129, 72, 100, "f32"),
    (1, 300, 256, 128, "bf16"), (3, 111, 124, 129, "f32"), (2, 128, 256, 130, "bf16")])
def test_backward(G, S, M, E, dt):
    shapes.test_random_shape(MoEConfig("dz", G=G, S=S, M=M, H=24, E=E, C=max(2, 3 * S // E), act_dtype=dt,
                                       seed=8800 + S + M + E))


@pytest.mark.parametrize("E,dt", [(100, "bf16"), (40, "f32"), (70, "f32")])
def test_training_step_captured_after_moe_prepare(E, dt):
    """Gates whose weight-gradient kernel takes more than 64 KB of LDS: moe_prepare is all the set-up that a
    captured step needs.  Every replay equals eager calls bit for bit."""
    cfg = MoEConfig("capture", G=2, S=192, M=136, H=72, E=E, C=8, act_dtype=dt, seed=70 + E)
    sh = shape_of(cfg)
    sets = [(make_inputs(cfg.with_(seed=cfg.seed + k), device=DEV), make_upstream(cfg.with_(seed=cfg.seed + k), device=DEV))
            for k in range(2)]
    live = [t.clone() for t in (sets[0][0].x, sets[0][0].wg, sets[0][0].u, sets[0][0].wi, sets[0][0].wo, *sets[0][1])]
    x, wg, u, wi, wo, dy, daux = live
    out = {"y": torch.empty_like(x), "aux": torch.empty(cfg.G, device=DEV), "dx": torch.empty_like(x),
           "dwg": torch.empty_like(wg), "dwi": torch.empty_like(wi), "dwo": torch.empty_like(wo)}
    fws = torch.empty(moe.moe_train_workspace_bytes(sh), dtype=torch.uint8, device=DEV)
    bws = torch.empty(moe.moe_backward_workspace_bytes(sh), dtype=torch.uint8, device=DEV)
    moe.moe_prepare()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        moe.moe_forward_train(sh, x, wg, u, wi, wo, out["y"], out["aux"], fws)
        moe.moe_backward(sh, x, wg, wi, wo, dy, daux, fws, out["dx"], out["dwg"], out["dwi"], out["dwo"], bws)
    for k in (1, 0, 1):
        inp, up = sets[k]
        for dst, src in zip(live, (inp.x, inp.wg, inp.u, inp.wi, inp.wo, *up)):
            dst.copy_(src)
        graph.replay()
        torch.cuda.synchronize()
        got = {name: t.clone() for name, t in out.items()}
        want = gpu_forward_backward(cfg, inp, *up)
        for name in got:
            assert torch.equal(got[name], want[name]), (k, name)
