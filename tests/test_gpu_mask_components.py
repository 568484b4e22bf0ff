"""Safety masks of stored trajectories read the components that carry a
constraint: first violations and least margins equal a float32 scan bit for
bit (each margin is one subtraction), whatever the other components hold."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_1906_02318_amd import mpmi

pytestmark = pytest.mark.gpu


# state sizes and boxed components; horizons around the chunk of four steps
@pytest.mark.parametrize("n,boxed", [(1, [0]), (2, [1]), (4, [0, 2]), (6, [4]), (6, [0, 5]), (8, [7]), (8, list(range(4)))])
@pytest.mark.parametrize("H", [1, 4, 7])
def test_unconstrained_components_are_not_part_of_the_verdict(n, boxed, H):
    rng = np.random.default_rng(10 * n + H)
    N = 301
    traj = rng.normal(0.0, 0.5, size=(H, n, N + 1)).astype(np.float32)
    for j in range(n):  # NaN and infinities: a violation where there is a box, nothing elsewhere
        traj[:, j].flat[rng.integers(traj[:, j].size, size=5)] = [np.nan, np.inf, -np.inf, 0.0, -0.0]
    sys = mpmi.linear_system(n, 1, [(k, 1.0, 0.125) for k in boxed], [-1.0], [1.0])
    ctx = mpmi.Context(0)
    model = mpmi.mpmi_model_pack(ctx, sys, torch.tensor(np.eye(n + 1, n), device="cuda"))
    fv, least = mpmi.safe_mask(ctx, model, torch.tensor(traj, device="cuda"))
    margin = np.min(np.float32(0.875) - np.abs(traj[:, boxed]), axis=1)  # NaN where one is
    want, low = np.full(N + 1, H + 1), np.full(N + 1, np.inf, dtype=np.float32)
    for s in range(H):
        going = want == H + 1
        low = np.where(going, np.where(np.isnan(margin[s]), margin[s], np.fmin(low, margin[s])), low)
        want[going & ~(margin[s] > 0)] = s + 1
    assert np.array_equal(fv.cpu().numpy(), want)
    assert np.array_equal(least.cpu().numpy(), low, equal_nan=True)
