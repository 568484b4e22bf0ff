"""Where the library leaves the several-lane forms of a basis given as data and
of the balance bot, read from the launch sizes of captured calls, and the same
decisions on both sides."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import synth
from paper_1906_02318_amd import mpmi
from tests import workloads as W
from tests.test_gpu_proposal_lanes import _launches

pytestmark = pytest.mark.gpu

PRECS = pytest.mark.parametrize("prec", [mpmi.PREC_FP32, mpmi.PREC_FP32_RECHECK64], ids=["fp32", "recheck64"])


def _dev(v):
    return torch.tensor(np.asarray(v), dtype=torch.float32, device="cuda")


def _tick(ctx, model, x, u, N, prec, block=0, H=12, one_lane=False):
    d = mpmi.tick_desc(N, H, gen=mpmi.GEN_UNIFORM, n_seg=2, seed=3, precision=prec, block=block)
    fv = torch.zeros(N + 1, dtype=torch.int16, device="cuda")
    out = torch.zeros(mpmi.SELECTION_BYTES, dtype=torch.uint8, device="cuda")
    traj = mpmi.new_traj(ctx, H, model.n, N + 1) if one_lane else None  # stored trajectories: one lane per candidate
    call = lambda: mpmi.mpmi_tick(ctx, model, d, x, u, out=out, first_violation=fv, traj=traj)  # noqa: E731
    call()
    torch.cuda.synchronize()
    return out, fv, call


def _described(ctx, D):
    """The first D features of the three-input car's basis, a slow drift as the operator."""
    tr = W.track_dict(W.rc_track())
    atoms, feats = synth.race_car3_basis()
    sys = mpmi.custom_system(6, 3, atoms, feats[:D], [(4, 2.0, 0.0)], synth.RC3_U_LO, synth.RC3_U_HI, track=tr,
                             eps32_box=[3e-4], eps32_track=2e-3)
    K = 1e-4 * np.random.default_rng(D).standard_normal((D, 6))
    for j in range(6):
        K[1 + j, j] += 1.0
    return mpmi.mpmi_model_pack(ctx, sys, torch.tensor(K, device="cuda"))


# candidates with the user's input on both sides of a limit: 48 features 65,537, 49 features 131,073
@PRECS
@pytest.mark.parametrize("D,count,lanes", [(10, 65537, 8), (10, 65538, 1), (48, 65537, 8), (48, 65538, 1),
                                           (49, 65538, 8), (49, 131073, 8), (49, 131074, 1)])
def test_described_bases(D, count, lanes, prec):
    ctx = mpmi.Context(0)
    model = _described(ctx, D)
    x, u = _dev(synth.race_car_states(1, W.rc_track(), seed=4)[0]), _dev([0.1, 0.2, -0.1])
    out, fv, call = _tick(ctx, model, x, u, count - 1, prec)
    assert _launches(call)[0] == ((count * lanes + 255) // 256, 256)
    one, fv1, _ = _tick(ctx, model, x, u, count - 1, prec, one_lane=True)
    assert torch.equal(out, one) and torch.equal(fv, fv1)


# workgroups of 512 above 32,768 candidates, of the size asked for where one is; a ragged last one
@PRECS
@pytest.mark.parametrize("track", [False, True])
@pytest.mark.parametrize("block,count,lanes,threads", [
    (0, 32768, 2, 256), (0, 32769, 2, 512), (0, 33025, 2, 512), (0, 70001, 2, 512), (0, 262145, 2, 512),
    (0, 262146, 1, 256), (256, 70001, 2, 256), (256, 262145, 2, 256), (256, 262146, 1, 256), (64, 65537, 2, 64), (64, 65538, 1, 64)])
def test_balance_bot(track, block, count, lanes, threads, prec):
    ctx = mpmi.Context(0)
    sys = mpmi.balance_bot_system(p_bound=0.5)
    if track:
        sys = mpmi._sys(mpmi.BASIS_BALANCE_BOT, 4, 1, [(2, 0.5, 0.0)], [-5.0], [5.0],
                        track=dict(r0=0.5, half=0.4, amp=[0.1, 0.05], freq=[3, 8], phase=[0.3, 1.0], infl=0.0),
                        eps32_box=[1e-4], eps32_track=1e-3)
    model = mpmi.mpmi_model_pack(ctx, sys, torch.tensor(W.bb_model()[0], device="cuda"))
    x, u = _dev([0.3, 0.2, 0.05, 0.3]), _dev([1.0])
    out, fv, call = _tick(ctx, model, x, u, count - 1, prec, block=block, H=40)
    assert _launches(call)[0] == ((count * lanes + threads - 1) // threads, threads)
    one, fv1, _ = _tick(ctx, model, x, u, count - 1, prec, H=40, one_lane=True)
    assert torch.equal(out, one) and torch.equal(fv, fv1)
    assert int((fv == 41).sum()) not in (0, count)  # verdicts on both sides
