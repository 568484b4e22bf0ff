"""The training pass at the edges of its blocks: one row, around a 32-row
block, around the stages and parts of the weight-gradient products and where
their tile and part sizes change, a batch whose last block belongs to a second
round of the workgroups, and the same gradient from a workspace that holds an
earlier batch's operands."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import synth
from oracle import mlp_oracle as M
from paper_1906_02318_amd import mpmi
from tests import workloads as W
from tests.test_gpu_mlp import BF16_U, GRAD_C, effective_params, gradient_error_scale, net_tensors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 31, 32, 33, 63, 65, 127, 129, 2047, 2049, 4095, 8193, 16385])
def test_gradient_and_forward_at_block_edges(B):
    rng = np.random.default_rng(B)
    X = np.concatenate([synth.race_car_states(B, W.rc_track(), seed=B + 1),
                        synth.uniform_user(B, synth.RC_U_LO, synth.RC_U_HI, seed=B + 2)], axis=1)
    X = X.astype(np.float32).astype(np.float64)
    T = rng.uniform(-0.95, 0.95, size=(B, 2)).astype(np.float32).astype(np.float64)
    mean, std = np.array([0.0, 0.0, 0.0, 10.0, 0.0, 0.0, 0.0, 0.0]), np.array([21.0, 21.0, 2.0, 3.0, 0.3, 0.2, 0.2, 1.7])
    mean, std = mean.astype(np.float32).astype(np.float64), std.astype(np.float32).astype(np.float64)
    flat = synth.mlp_init(6) + 0.02 * rng.standard_normal(mpmi.MLP_PARAMS)
    ctx = mpmi.Context(0)
    net = net_tensors(flat, mean, std)
    Xd, Td = (torch.tensor(v, dtype=torch.float32, device="cuda") for v in (X, T))
    args = (ctx, net["w16"], net["w32"], net["mean"], net["std"], Xd)
    # A workspace last used by a larger batch: nothing of it may show.
    work = mpmi.mlp_workspace(ctx, B + 40)
    junk = torch.randn((B + 40, 8), device="cuda")
    mpmi.mlp_grad(*args[:5], junk, junk[:, :2].contiguous(), work=work)
    grad, loss = mpmi.mlp_grad(*args, Td, work=work)
    fresh, _ = mpmi.mlp_grad(*args, Td)
    assert torch.equal(grad, fresh)  # fixed-order sums
    eff = effective_params(flat)
    Lo, go = M.loss_and_grad(eff, X, T, mean, std)
    R = gradient_error_scale(eff, X, T, mean, std)
    # As in test_mlp_gradient_parity: GRAD_C BF16 roundings per term, their signs independent.  That
    # bound is one of sums over samples; a single sample keeps the whole vector's.
    g = grad.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(g - go) <= 6e-2 * np.linalg.norm(go)
    if B > 1:
        assert np.all(np.abs(g - go) <= GRAD_C * BF16_U * np.maximum(R, 1e-30))
    assert abs(loss.item() - Lo) <= 2e-2 * max(1.0, abs(Lo))
    Y = mpmi.mlp_forward(*args).cpu().numpy()
    Yo, _ = M.forward(eff, X, mean, std)
    assert np.abs(Y - Yo).max() <= 3e-2 * np.sqrt(np.mean(Yo ** 2))
