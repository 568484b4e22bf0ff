"""A lifted race-car tick's first violations do not depend on the batch: ragged
counts around the 16-candidate tile, the 64-candidate wave and the
256-candidate pass equal the same candidates in a batch of more passes than
workgroups, bit for bit; states from which tiles end early and states from
which none does, with and without stored states."""
from __future__ import annotations

import pytest
import torch

import synth
from paper_1906_02318_amd import mpmi
from tests import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [1, 13, 60])
@pytest.mark.parametrize("seed", [3, 4])
def test_ragged_batches_agree_with_a_large_one(H, seed):
    ctx = mpmi.Context(0)
    K, KL = W.rc_model()[0], W.rc_lifted_model()[0]
    model = mpmi.mpmi_model_pack(ctx, mpmi.race_car_system(W.track_dict(W.rc_track())), torch.tensor(K, device="cuda"))
    lifted = mpmi.mpmi_lifted_pack(ctx, model, torch.tensor(KL, device="cuda"), 60)
    x = torch.tensor(synth.race_car_states(1, W.rc_track(), seed=seed)[0], dtype=torch.float32, device="cuda")
    u = torch.tensor(synth.uniform_user(1, synth.RC_U_LO, synth.RC_U_HI, seed=seed)[0], dtype=torch.float32, device="cuda")

    def tick(N, store=False):
        fv = torch.zeros(N + 1, dtype=torch.int16, device="cuda")
        traj = mpmi.new_traj(ctx, H, model.n, N + 1) if store else None
        rec = mpmi.mpmi_tick_lifted(ctx, lifted, mpmi.tick_desc(N, H, gen=mpmi.GEN_UNIFORM, seed=9, tick=seed), x, u,
                                    first_violation=fv, traj=traj)
        return mpmi.decode_selection(rec), fv

    _, whole = tick(600000)
    for N in (0, 14, 15, 16, 62, 63, 64, 255, 256, 1000):
        for store in (False, True):
            sel, fv = tick(N, store)
            assert torch.equal(fv, whole[:N + 1]), (N, store)
            assert sel["n_safe"] == int((fv[1:] == H + 1).sum()), (N, store)
