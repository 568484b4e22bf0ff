"""The forms a tick takes by itself: whatever number of lanes per candidate
the library picks (counts on both sides of its limits, FP32 and
FP32_RECHECK64, custom bases of every feature and atom count class), the
record and the first violations are those of the one-lane form, which a
trajectory store or a workgroup of 512 selects."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import synth
from paper_1906_02318_amd import mpmi
from tests import workloads as W

pytestmark = pytest.mark.gpu


def _tick(ctx, model, x, u, one_lane, prec, gen, N, H, S, grid=None, cand=None, tick=0):
    """(record, first violations); the one-lane form of a custom basis is the one that stores trajectories."""
    fv = torch.zeros(N + 1, dtype=torch.int16, device="cuda")
    custom = model.system.basis == mpmi.BASIS_CUSTOM
    d = mpmi.tick_desc(N, H, gen=gen, grid=grid, n_seg=S, seed=3, tick=tick, precision=prec,
                       block=512 if one_lane and not custom else 0)
    traj = mpmi.new_traj(ctx, H, model.n, N + 1) if one_lane and custom else None
    rec = mpmi.mpmi_tick(ctx, model, d, x, u, cand=cand, first_violation=fv, traj=traj)
    return rec, fv


def _same(ctx, model, x, u, *args, **kw):
    a, b = _tick(ctx, model, x, u, True, *args, **kw), _tick(ctx, model, x, u, False, *args, **kw)
    assert torch.equal(a[0], b[0]), (mpmi.decode_selection(a[0]), mpmi.decode_selection(b[0]))
    assert torch.equal(a[1], b[1])


def _dev(v):
    return torch.tensor(np.asarray(v), dtype=torch.float32, device="cuda")


@pytest.mark.parametrize("prec", [mpmi.PREC_FP32, mpmi.PREC_FP32_RECHECK64], ids=["fp32", "recheck64"])
@pytest.mark.parametrize("kind,N", [("bb", 0), ("bb", 63), ("bb", 4096), ("bb", 4097), ("bb", 262145), ("rc", 1),
                                    ("rc", 8191), ("rc", 8192), ("rc", 16383), ("rc", 16384), ("rc", 32768),
                                    ("rc", 32900), ("rc", 49152), ("bb", 8191), ("bb", 8192), ("rc", 16448),
                                    ("rc", 32767), ("rc", 49151), ("rc", 65535), ("rc", 65536)])
def test_fixed_bases_take_the_same_decision_in_every_form(prec, kind, N):
    ctx = mpmi.Context(0)
    if kind == "bb":
        model = mpmi.mpmi_model_pack(ctx, mpmi.balance_bot_system(), torch.tensor(W.bb_model()[0], device="cuda"))
        states, lo, hi, S = synth.balance_bot_states(3, seed=4), [-5.0], [5.0], 5
    else:
        model = mpmi.mpmi_model_pack(ctx, mpmi.race_car_system(W.track_dict(W.rc_track())),
                                     torch.tensor(W.rc_model()[0], device="cuda"))
        states, lo, hi, S = synth.race_car_states(3, W.rc_track(), seed=4), synth.RC_U_LO, synth.RC_U_HI, 2
    users = synth.uniform_user(3, lo, hi, seed=5)
    for i in range(3):
        _same(ctx, model, _dev(states[i]), _dev(users[i]), prec, mpmi.GEN_UNIFORM, N, 37, S, tick=i)
    # two boxes on one component, one without a box, no track: the rounding band's and the limits' other cases
    if kind == "bb":
        sys = mpmi.balance_bot_system()
        sys.n_box = 3
        sys.box_index[2], sys.box_bound[2], sys.eps32_box[2] = 2, 0.3, 2e-4
        model = mpmi.mpmi_model_pack(ctx, sys, torch.tensor(W.bb_model()[0], device="cuda"))
        _same(ctx, model, _dev(states[0]), _dev(users[0]), prec, mpmi.GEN_UNIFORM, N, 21, 1)


@pytest.mark.parametrize("prec", [mpmi.PREC_FP32, mpmi.PREC_FP32_RECHECK64], ids=["fp32", "recheck64"])
@pytest.mark.parametrize("D,n,m,track", [(1, 1, 1, False), (7, 3, 2, True), (8, 2, 1, True), (9, 6, 3, True),
                                         (31, 8, 4, True), (32, 5, 1, False), (33, 6, 2, True), (63, 7, 4, True),
                                         (64, 6, 3, True), (64, 8, 4, False)])
def test_custom_bases_take_the_same_decision_in_both_forms(prec, D, n, m, track):
    """Random stable-ish operators on bases of 1 .. 32 atoms; limits put verdicts on both sides."""
    rng = np.random.default_rng(100 * D + 10 * n + m)
    nw = n + m
    atoms = [("one", 0)] + [("var", k) for k in range(nw)] + [("sin", k) for k in range(nw)] + \
        [("cos", k) for k in range(nw)]
    atoms = atoms[:32] if D >= 31 else atoms[:1 + nw]
    feats = [(1 + k, 0) for k in range(nw)]
    while len(feats) < D:
        feats.append((int(rng.integers(len(atoms))), int(rng.integers(len(atoms)))))
    feats = feats[:D]
    box = [(k, 1.5, 0.0) for k in range(min(4, n))]
    tr = dict(r0=1.0, half=0.8, amp=[0.1, 0.05], freq=[3, 8], phase=[0.3, 1.0], infl=0.0) if track else None
    sys = mpmi.custom_system(n, m, atoms, feats, box, [-1.0] * m, [1.0] * m, track=tr, eps32_box=[1e-3] * len(box),
                             eps32_track=1e-3)
    K = 0.03 * rng.standard_normal((D, n))
    for j in range(min(n, D)):
        K[j, j] += 0.99
    ctx = mpmi.Context(0)
    model = mpmi.mpmi_model_pack(ctx, sys, torch.tensor(K, device="cuda"))
    x = 0.4 * rng.standard_normal(n)
    if track:
        x[:2] = 0.7, 0.7
    u = rng.uniform(-1.0, 1.0, size=m)
    for N, H, S in ((0, 3, 1), (1000, 40, 1), (2049, 25, 3)):
        cand = torch.tensor(rng.uniform(-1.0, 1.0, size=(S, m, max(N, 1))), dtype=torch.float32, device="cuda")
        _same(ctx, model, _dev(x), _dev(u), prec, mpmi.GEN_EXPLICIT, N, H, S, cand=cand)


def test_rules_leave_the_other_calls_as_they_were():
    """Process noise, a linear basis and stored trajectories keep the one-lane form; refused requests stay refused."""
    ctx = mpmi.Context(0)
    K = torch.tensor(W.bb_model()[0], device="cuda")
    noisy = mpmi.mpmi_model_pack(ctx, mpmi.balance_bot_system(noise=[1e-3, 0.0, 1e-3, 0.0]), K)
    x, u = _dev(synth.balance_bot_states(1, seed=4)[0]), _dev([1.0])
    _same(ctx, noisy, x, u, mpmi.PREC_FP32, mpmi.GEN_UNIFORM, 2000, 30, 1)
    plain = mpmi.mpmi_model_pack(ctx, mpmi.balance_bot_system(), K)
    with pytest.raises(mpmi.MpmiError):
        mpmi.mpmi_tick(ctx, plain, mpmi.tick_desc(100, 10, grid=[100], lanes_per_cand=4,
                                                  precision=mpmi.PREC_FP32_RECHECK64), x, u)
    lin = mpmi.mpmi_model_pack(ctx, mpmi.linear_system(4, 1, [(0, 2.0, 0.0)], [-5.0], [5.0]),
                               torch.tensor(0.1 * np.eye(5, 4) + 0.01, device="cuda"))
    _same(ctx, lin, x, u, mpmi.PREC_FP32, mpmi.GEN_UNIFORM, 300, 20, 1)
