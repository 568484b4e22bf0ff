"""The number of lanes that the library picks for the race car on both sides of
16,384 candidates, read from the launch sizes of captured calls."""
from __future__ import annotations

import pytest
import torch

import synth
from paper_1906_02318_amd import mpmi
from tests import workloads as W
from tests.test_gpu_proposal_lanes import _launches

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def car():
    ctx = mpmi.Context(0)
    model = mpmi.mpmi_model_pack(ctx, mpmi.race_car_system(W.track_dict(W.rc_track())),
                                 torch.tensor(W.rc_model()[0], device="cuda"))
    x = torch.tensor(synth.race_car_states(1, W.rc_track(), seed=4)[0], dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    return ctx, model, x


# candidates with the user's input: 16,384, 16,385 and 16,386
@pytest.mark.parametrize("N,lanes", [(16383, 4), (16384, 4), (16385, 2)])
def test_tick(car, N, lanes):
    ctx, model, x = car
    u, out = torch.zeros(2, device="cuda"), torch.zeros(mpmi.SELECTION_BYTES, dtype=torch.uint8, device="cuda")
    d = mpmi.tick_desc(N, 20, gen=mpmi.GEN_UNIFORM)
    mpmi.mpmi_tick(ctx, model, d, x, u, out=out)
    assert _launches(lambda: mpmi.mpmi_tick(ctx, model, d, x, u, out=out)) == [(((N + 1) * lanes + 255) // 256, 256)]


@pytest.mark.parametrize("Nc,lanes", [(16384, 4), (16385, 2)])
def test_stored_rollout(car, Nc, lanes):
    ctx, model, x = car
    cand, traj = torch.zeros((1, 2, Nc), device="cuda"), mpmi.new_traj(ctx, 20, 6, Nc)
    mpmi.rollout_batch(ctx, model, x, cand, 20, traj=traj)
    assert _launches(lambda: mpmi.rollout_batch(ctx, model, x, cand, 20, traj=traj)) == [((Nc * lanes + 255) // 256, 256)]
