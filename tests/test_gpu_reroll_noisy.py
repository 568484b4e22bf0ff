"""The FP64 re-roll of noisy described bases: a row of lanes per kept candidate up
to 24,576, one lane in a launch of its own above.  Whole lists on both sides
against the many-loop form, and replays of a captured tick whose list is now
long, now short, now empty."""
from __future__ import annotations

import pytest
import torch

import synth
from paper_1906_02318_amd import mpmi
from tests import workloads as W
from tests.test_gpu_proposal_lanes import _launches
from tests.test_gpu_reroll_rows import _against_the_many_loop_form

pytestmark = pytest.mark.gpu
NOISE = [1e-3, 0.0, 2e-3, 1e-3]


def _model(ctx, eps, track=False):
    sys = mpmi.balance_bot_system(eps32=(eps, eps), noise=NOISE)
    if track:  # degree 8: the other instance
        sys = mpmi._sys(mpmi.BASIS_BALANCE_BOT, 4, 1, [(2, 0.5, 0.0)], [-5.0], [5.0], noise=NOISE,
                        track=dict(r0=0.5, half=0.4, amp=[0.1, 0.05], freq=[3, 8], phase=[0.3, 1.0], infl=0.0),
                        eps32_box=[eps], eps32_track=eps)
    return mpmi.mpmi_model_pack(ctx, sys, torch.tensor(W.bb_model()[0], device="cuda"))


# entries = N + 1
@pytest.mark.parametrize("N,track", [(24574, False), (24575, False), (24575, True), (24576, False), (24576, True),
                                     (40001, False)])
def test_whole_lists(N, track):
    ctx = mpmi.Context(0)
    states = synth.balance_bot_states(3, seed=23)
    if track:
        states[:, :2] = 0.3, 0.4
    _against_the_many_loop_form(ctx, _model(ctx, 1e30, track), states,
                                synth.uniform_user(3, [-5.0], [5.0], seed=24), N, 15, 2)


@pytest.mark.parametrize("N,launches", [(24575, 3), (24576, 4)])
def test_replays(N, launches):
    ctx = mpmi.Context(0)
    model, wide = _model(ctx, 1e-3), _model(ctx, 1e30)
    x, u = torch.zeros(4, device="cuda"), torch.zeros(1, device="cuda")
    d = mpmi.tick_desc(N, 15, gen=mpmi.GEN_GRID, grid=[N], n_seg=1, precision=mpmi.PREC_FP32_RECHECK64)
    out = torch.zeros(mpmi.SELECTION_BYTES, dtype=torch.uint8, device="cuda")
    fv = torch.zeros(N + 1, dtype=torch.int16, device="cuda")
    mpmi.mpmi_tick(ctx, model, d, x, u, out=out, first_violation=fv)
    assert len(_launches(lambda: mpmi.mpmi_tick(ctx, model, d, x, u, out=out, first_violation=fv))) == launches
    graphs = [(m, mpmi.TickGraph(ctx, m, d, x, u, out=out, first_violation=fv)) for m in (wide, model)]
    kept = []
    for i, state in enumerate(synth.balance_bot_states(3, seed=5).tolist() + [[9.0, 0.0, 0.0, 0.0]]):
        x.copy_(torch.tensor(state))
        u.fill_(0.5 * i)
        for m, g in graphs:
            g.launch()
            torch.cuda.synchronize()
            got, got_fv = out.clone(), fv.clone()
            kept.append(mpmi.decode_selection(got)["n_recheck"])
            mpmi.mpmi_tick(ctx, m, d, x, u, out=out, first_violation=fv)
            torch.cuda.synchronize()
            assert torch.equal(got, out) and torch.equal(got_fv, fv)
    assert max(kept) == N + 1 and min(kept) == 0
