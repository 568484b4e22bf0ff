"""The Gram kernel's instances of one, two and four column blocks, against
NumPy's least squares: state and input as the features (3 and 12) over several
tiles per workgroup, and described bases at the widest of one and two blocks."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_1906_02318_amd import mpmi
from tests.test_gpu_fit_blocks import _basis, _lift

pytestmark = pytest.mark.gpu


def _check(sys, P, PY, X, U, Y):
    D, s = P.shape[1], np.sqrt(np.mean(P * P, axis=0))
    sv = np.linalg.svd(P / s, compute_uv=False)
    cond = sv[0] / sv[-1]
    ctx = mpmi.Context(0)
    d = [torch.tensor(v, device="cuda") for v in (X, U, Y)]
    for fit, target in ((mpmi.koopman_fit, Y), (mpmi.koopman_fit_lifted, PY)):
        K, _ = fit(ctx, sys, *d)
        want = np.linalg.lstsq(P / s, target, rcond=None)[0]
        # Normal equations: backward error of order D eps in the Gram matrix, amplified by cond^2.
        tol = 20 * D * np.finfo(np.float64).eps * cond ** 2 * np.linalg.norm(want)
        assert np.linalg.norm(K.cpu().numpy() * s[:, None] - want) <= max(tol, 1e-13)


@pytest.mark.parametrize("n,m,T", [(2, 1, 40), (2, 1, 70000), (8, 4, 16385), (1, 1, 64)])
def test_state_and_input_as_features(n, m, T):
    rng = np.random.default_rng(100 * n + T)
    X, U, Y = (rng.uniform(-2.0, 2.0, size=(T, k)) for k in (n, m, n))
    sys = mpmi.linear_system(n, m, [(0, 1.0, 0.0)], [-2.0] * m, [2.0] * m)
    _check(sys, np.concatenate([X, U], axis=1), np.concatenate([Y, U], axis=1), X, U, Y)


@pytest.mark.parametrize("D", [16, 17, 32, 33])
def test_described_bases(D):
    T = 33000
    rng = np.random.default_rng(D)
    X, U, Y = (rng.uniform(-2.0, 2.0, size=(T, k)) for k in (6, 2, 6))
    atoms, feats = _basis(D)
    sys = mpmi.custom_system(6, 2, atoms, feats, [], (-2.0, -2.0), (2.0, 2.0))
    _check(sys, _lift(atoms, feats, np.concatenate([X, U], axis=1)), _lift(atoms, feats, np.concatenate([Y, U], axis=1)),
           X, U, Y)
