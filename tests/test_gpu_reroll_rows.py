"""The race car's FP64 re-roll over a whole list: bands so wide that every
candidate is listed and nothing precedes the list, so every first violation
is the re-roll's.  Against the many-loop form, which predicts one candidate
per lane.  The two add the same terms in other orders, so a verdict could
differ only where a margin is within some 1e-13 of zero; over the at most
8,193 x 60 margins of a case, of spread about one, that is a chance of 1e-7."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import synth
from paper_1906_02318_amd import mpmi
from tests import workloads as W

pytestmark = pytest.mark.gpu


def _turning_model():
    """x' = x but for: psi' = psi + 1 + delta / 10, vy' = vy + cos(psi) / 20, X' = X + sin(psi) / 1000."""
    K = np.zeros_like(W.rc_model()[0])
    K[1 + np.arange(6), np.arange(6)] = 1.0
    K[0, 2], K[7, 2], K[46, 4], K[45, 0] = 1.0, 0.1, 0.05, 1e-3
    return K


# entries = N + 1: one, a row short of a wave, a wave, one over, and both sides of the 16-lane form's limit
@pytest.mark.parametrize("N,H,S,psi,noise", [(1, 7, 1, None, False), (2, 60, 3, None, False), (3, 60, 8, None, False),
                                             (4, 5, 8, None, False), (260, 60, 7, None, True),
                                             (8191, 60, 2, None, False), (8192, 60, 2, None, False),
                                             (70, 40, 4, 2.0 ** 20 - 20, False), (8192, 40, 4, 2.0 ** 20 - 20, False),
                                             (9, 12, 1, 3e6, False)])
def test_every_first_violation_is_the_one_lane_forms(N, H, S, psi, noise):
    ctx = mpmi.Context(0)
    sys = mpmi.race_car_system(W.track_dict(W.rc_track()), eps32_track=1e30, eps32_vy=1e30,
                               noise=[1e-3, 0.0, 1e-4, 0.0, 2e-3, 1e-3] if noise else None)
    K = W.rc_model()[0] if psi is None else _turning_model()
    model = mpmi.mpmi_model_pack(ctx, sys, torch.tensor(K, device="cuda"))
    states, users = synth.race_car_states(3, W.rc_track(), seed=21), synth.uniform_user(
        3, synth.RC_U_LO, synth.RC_U_HI, seed=22)
    for i in range(3):
        x = torch.tensor(states[i], dtype=torch.float32, device="cuda")
        if psi is not None:
            x[2] = psi
        u = torch.tensor(users[i], dtype=torch.float32, device="cuda")
        fv = torch.zeros(N + 1, dtype=torch.int16, device="cuda")
        rec = mpmi.mpmi_tick(ctx, model, mpmi.tick_desc(N, H, gen=mpmi.GEN_UNIFORM, n_seg=S, seed=5, tick=i,
                                                        precision=mpmi.PREC_FP32_RECHECK64), x, u, first_violation=fv)
        loop = dict(model=model, x_t=x, u_user=u, n_cand=N, horizon=H, gen=mpmi.GEN_UNIFORM, n_seg=S, seed=5, tick=i,
                    out=torch.zeros(mpmi.SELECTION_BYTES, dtype=torch.uint8, device="cuda"),
                    first_violation=torch.zeros(N + 1, dtype=torch.int16, device="cuda"))
        multi = mpmi.Multi(ctx, [loop], block=256, precision=mpmi.PREC_FP32_RECHECK64)
        try:
            multi.tick()
            torch.cuda.synchronize()
        finally:
            multi.close()
        assert mpmi.decode_selection(rec)["n_recheck"] == N + 1
        assert torch.equal(fv, loop["first_violation"])
        assert torch.equal(rec, loop["out"])
