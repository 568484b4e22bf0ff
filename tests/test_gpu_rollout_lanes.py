"""A stored rollout's states do not depend on the number of lanes the library
gives a candidate: every batch size on both sides of its limits, against the
same candidates inside a batch large enough for one lane each, bit for bit."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import synth
from paper_1906_02318_amd import mpmi
from tests import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,S", [(1, 1), (13, 3), (5, 8)])
@pytest.mark.parametrize("kind,sizes", [("rc", (1, 63, 8192, 8193, 16448, 16449, 32768, 32769, 65536)),
                                        ("bb", (1, 255, 32768, 32769, 65536))])
def test_small_batches_store_the_large_batchs_states(kind, sizes, H, S):
    ctx = mpmi.Context(0)
    if kind == "bb":
        sys, K, x0, lo, hi = mpmi.balance_bot_system(), W.bb_model()[0], synth.balance_bot_states(1, seed=8)[0], [-5.0], [5.0]
    else:
        sys, K = mpmi.race_car_system(W.track_dict(W.rc_track())), W.rc_model()[0]
        x0, lo, hi = synth.race_car_states(1, W.rc_track(), seed=8)[0], synth.RC_U_LO, synth.RC_U_HI
    model = mpmi.mpmi_model_pack(ctx, sys, torch.tensor(K, device="cuda"))
    x0 = torch.tensor(x0, dtype=torch.float32, device="cuda")
    big = 70000
    rng = np.random.default_rng(H + S)
    lo, hi = np.asarray(lo).reshape(1, -1, 1), np.asarray(hi).reshape(1, -1, 1)
    cand = torch.tensor(rng.uniform(lo, hi, size=(S, lo.size, big)), dtype=torch.float32, device="cuda")
    whole = mpmi.rollout_batch(ctx, model, x0, cand, H)
    for n in sizes:
        part = mpmi.rollout_batch(ctx, model, x0, cand[:, :, big - n:].contiguous(), H)
        assert torch.equal(part.contiguous().view(torch.int32), whole[:, :, big - n:].contiguous().view(torch.int32)), n
