"""The data and the weight gradient of a linear layer in one launch.  moe_backward_events, which marks each product, launches
them one after the other with the same arithmetic: every gradient equal bit for bit, at the edges of the tiles of the nine
pairs, and with the weights' own memory as that of their gradients.  Which pair each case takes is pinned by
test_kernel_rules.py."""
import pytest
import torch

import paper_2006_16668_amd as moe
from harness import shape_of
from paper_2006_16668_amd.binding import BACKWARD_EVENTS
from workloads import MoEConfig, make_inputs, make_upstream

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _cfg(G, S, M, H, E, C, bias=0.0):
    return MoEConfig(f"G{G}_S{S}_M{M}_H{H}_E{E}_C{C}", G=G, S=S, M=M, H=H, E=E, C=C, act_dtype="bf16", seed=4100 + M + H + E,
                     logit_bias_std=bias)


CASES = [
    _cfg(1, 40, 128, 8, 3, 1),                     # one row per expert, one step
    _cfg(5, 60, 328, 72, 3, 13),                   # 64 x 64, tails of rows, columns and k
    _cfg(1, 130, 64, 64, 2, 64),                   # whole tiles
    _cfg(4, 22, 768, 1536, 4, 11),                 # long sums of few tiles
    _cfg(2, 300, 384, 1032, 100, 6, 0.5),          # weights of 128 x 128, few rows, empty experts
    _cfg(3, 200, 768, 3072, 23, 18),
    _cfg(2, 2120, 216, 440, 18, 236, 1.0),         # 64 x 128
    _cfg(1, 3000, 256, 512, 6, 1000),              # 128 x 128 rows
    _cfg(4, 627, 800, 3232, 46, 28),
    _cfg(2, 1500, 136, 904, 24, 195, 0.5),
    _cfg(4, 1024, 512, 2048, 16, 128, 0.5),        # dh of the persistent kernel, with its mask bits, when alone
    _cfg(2, 1318, 512, 2048, 9, 293),
    _cfg(8, 595, 168, 504, 99, 13),                # 128 x 128 rows beside weights of 64 x 64 tiles
    _cfg(1, 3464, 256, 1024, 21, 330),             # and of 64 x 128
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_one_launch_equals_two(cfg):
    print(cfg, flush=True)
    sh = shape_of(cfg)
    inp = make_inputs(cfg, device=DEV)
    dy, daux = make_upstream(cfg, device=DEV)
    y, aux = torch.empty_like(inp.x), torch.empty(cfg.G, device=DEV)
    fws = torch.empty(moe.moe_train_workspace_bytes(sh), dtype=torch.uint8, device=DEV)
    moe.moe_forward_train(sh, inp.x, inp.wg, inp.u, inp.wi, inp.wo, y, aux, fws)

    def backward(call, in_place, *extra):
        wi, wo = inp.wi.clone(), inp.wo.clone()
        out = [torch.full_like(t, float("nan")) for t in (inp.x, inp.wg)]
        out += [wi, wo] if in_place else [torch.full_like(t, float("nan")) for t in (wi, wo)]
        ws = torch.empty(moe.moe_backward_workspace_bytes(sh), dtype=torch.uint8, device=DEV)
        call(sh, inp.x, inp.wg, wi, wo, dy, daux, fws, *out, ws, *extra)
        torch.cuda.synchronize()
        return out

    events = [torch.cuda.Event(enable_timing=True) for _ in range(BACKWARD_EVENTS)]
    for e in events:
        e.record()
    want = backward(moe.moe_backward_events, False, events)
    for in_place in (False, True):
        for name, g, w in zip(("dx", "dwg", "dwi", "dwo"), backward(moe.moe_backward, in_place), want):
            assert torch.isfinite(g.float()).all(), name
            assert torch.equal(g, w), (name, in_place)
