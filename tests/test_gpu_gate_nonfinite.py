"""Tokens whose row of x holds infinities or NaN, in every gate kernel: their choices are valid expert
indices, two different ones, positions are counted as for any token, and no other token's choices or
rows of y change.  fp32: an infinite feature makes logits of both signs, ranked as infinities are."""
import numpy as np
import pytest
import torch

from harness import gpu_forward, gpu_gate
from oracle import moe_oracle as orc
from workloads import MoEConfig, make_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
INF, NAN = float("inf"), float("nan")


def _positions(idx, not_sampled, E, C):
    """Slots and fill that Algorithm 1 gives these choices: first choices in token order, then second ones."""
    S = idx.shape[0]
    slot = np.full((S, 2), -2)
    count = np.zeros(E, dtype=int)
    for k in range(2):
        for s in range(S):
            if k == 0 or not not_sampled[s]:
                slot[s, k] = count[idx[s, k]] if count[idx[s, k]] < C else -1
                count[idx[s, k]] += 1
    return slot, np.minimum(count, C)


@pytest.mark.parametrize("G,S,M,E,C,dt", [
    (1, 60, 36, 4, 40, "f32"), (2, 130, 64, 2, 90, "f32"), (1, 200, 136, 100, 5, "f32"), (1, 70, 64, 130, 3, "f32"),
    (1, 64, 128, 8, 20, "bf16"), (3, 100, 136, 40, 9, "bf16"), (300, 64, 64, 5, 30, "bf16"), (260, 66, 72, 33, 8, "bf16"),
    (1, 200, 136, 100, 5, "bf16"), (1, 90, 72, 300, 2, "bf16"), (1, 70, 64, 600, 2, "bf16"), (1, 256, 128, 600, 2, "bf16")])
def test_choices_stay_valid(G, S, M, E, C, dt):
    print(f"G={G} S={S} M={M} E={E} C={C} {dt}", flush=True)
    cfg = MoEConfig("nonfinite", G=G, S=S, M=M, H=72, E=E, C=C, act_dtype=dt, seed=900 + S + M + E)
    inp = make_inputs(cfg, device=DEV)
    inp.wg[M - 1] = -inp.wg[M - 1].abs() - 1e-3            # a feature that counts against every expert
    bad = {3: (slice(None), NAN), 7: (0, INF), 8: (0, -INF), 20: (slice(None), INF), 33: (M - 1, INF), S - 1: (M // 2, NAN)}
    touched = np.zeros((G, S), dtype=bool)
    inp.x[:, :, M - 1] = 0                                 # (only infinities meet it)
    clean_x = inp.x.to("cpu", torch.float64).numpy()
    gates = orc.softmax_gates(clean_x, inp.wg.to("cpu", torch.float64).numpy())
    z = np.sort(gates, axis=-1)
    sure = (z[..., -1] > z[..., -2] * 1.001) & (z[..., -2] > z[..., -3] * 1.001 if E > 2 else True)
    clean = orc.top2_gating(gates, inp.u.to("cpu", torch.float64).numpy(), C)["expert_idx"]
    for s, (where, v) in bad.items():
        inp.x[G - 1, s, where] = v
        touched[G - 1, s] = True
    r = gpu_gate(cfg, inp.x, inp.wg, inp.u)
    idx, slot = r["expert_idx"].cpu().numpy(), r["slot"].cpu().numpy()
    assert idx.min() >= 0 and idx.max() < E and (idx[..., 0] != idx[..., 1]).all()
    keep = sure & ~touched
    assert keep.sum() > 0.9 * G * S - 6 and (idx[keep] == clean[keep]).all()
    for g in {0, G - 1}:
        want, fill = _positions(idx[g], slot[g, :, 1] == -2, E, C)
        assert (slot[g] == want).all() and (r["fill"][g].cpu().numpy() == fill).all()
    if dt == "f32" and E <= 128:
        wg = inp.wg.cpu().numpy()
        for s, sign in ((7, 1), (8, -1)):                  # logits of one infinity: +inf first, lowest index first
            order = np.concatenate([np.flatnonzero(sign * wg[0] > 0), np.flatnonzero(sign * wg[0] < 0)])
            assert (idx[G - 1, s] == order[:2]).all(), (s, idx[G - 1, s], order[:2])
        assert (idx[G - 1, 33] == [0, 1]).all()            # -inf for every expert
    if M >= 128 or G < 10:
        y, _ = gpu_forward(cfg, inp)
        assert np.isfinite(y.float().cpu().numpy()[~touched]).all()
