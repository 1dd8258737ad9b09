"""The kernel that forms dout, the dispatched rows and the gradient of the gate logits: a wavefront per token, and blocks that
clear the rows no token fills.  The workspace is full of NaN before, so a row that is neither formed nor cleared reaches the
weight gradients.  Gradients against the oracle within the tolerances of the drawn shapes."""
import numpy as np
import pytest
import torch

import paper_2006_16668_amd as moe
from harness import f64, rel_fro, shape_of
from oracle import moe_oracle_backward as orb
from workloads import ExpertWeightsF64, MoEConfig, make_inputs, make_upstream

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _cfg(dt, G, S, M, H, E, C, bias=0.0):
    return MoEConfig(f"{dt}_G{G}_S{S}_M{M}_H{H}_E{E}_C{C}", G=G, S=S, M=M, H=H, E=E, C=C, act_dtype=dt,
                     seed=5200 + G * S + M + E, logit_bias_std=bias)


CASES = [
    _cfg("f32", 1, 17, 8, 8, 2, 3),                    # one piece of a row; most choices dropped
    _cfg("f32", 3, 43, 264, 40, 7, 64, 1.0),           # rows of two rounds of a wavefront; many empty rows
    _cfg("f32", 2, 33, 776, 40, 5, 16, 0.5),           # of three rounds, taken two at a time, and a bit
    _cfg("bf16", 1, 65, 512, 64, 3, 63),
    _cfg("bf16", 2, 64, 520, 64, 16, 32, 1.0),         # one lane more than a row of 512; empty experts' rows
    _cfg("bf16", 5, 51, 72, 136, 33, 13),              # 255 tokens, more gate columns than half a wavefront
    _cfg("bf16", 4, 100, 128, 72, 65, 16, 0.5),        # more gate columns than a wavefront
    _cfg("bf16", 2, 128, 256, 256, 129, 8, 0.5),       # dz in three bf16 terms
    _cfg("bf16", 2, 700, 256, 512, 4, 256, 1.0),       # packed rows, 256-row tiles partly full
    _cfg("bf16", 1, 300, 256, 256, 3, 256, 2.0),       # packed rows, one expert nearly empty
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_gradients_from_a_used_workspace(cfg):
    print(cfg, flush=True)
    sh = shape_of(cfg)
    inp = make_inputs(cfg, device=DEV)
    dy, daux = make_upstream(cfg, device=DEV)
    x, wg, u = inp.host_f64()
    want = orb.moe_backward(x, wg, u, ExpertWeightsF64(inp.wi), ExpertWeightsF64(inp.wo), cfg.C, f64(dy), f64(daux))
    y, aux = torch.empty_like(inp.x), torch.empty(cfg.G, device=DEV)
    fws = torch.empty(moe.moe_train_workspace_bytes(sh), dtype=torch.uint8, device=DEV)
    moe.moe_forward_train(sh, inp.x, inp.wg, inp.u, inp.wi, inp.wo, y, aux, fws)
    ws = torch.full((moe.moe_backward_workspace_bytes(sh),), 255, dtype=torch.uint8, device=DEV)
    got = {k: torch.full_like(t, float("nan")) for k, t in
           (("dx", inp.x), ("dwg", inp.wg), ("dwi", inp.wi), ("dwo", inp.wo))}
    moe.moe_backward(sh, inp.x, inp.wg, inp.wi, inp.wo, dy, daux, fws, *got.values(), ws)
    torch.cuda.synchronize()
    tol = 2e-2 if cfg.act_dtype == "bf16" else 2e-5
    for k, v in got.items():
        ref = np.stack([want[k][e] for e in range(cfg.E)]) if k in ("dwi", "dwo") else want[k]
        assert torch.isfinite(v.float()).all(), k
        assert rel_fro(f64(v), ref) < tol, k
