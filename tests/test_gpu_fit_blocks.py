"""The FP64 fit at the edges of its 16-wide blocks and 64-row tiles, against
NumPy's least squares: feature counts around multiples of 16, row counts around
a tile and around one tile per workgroup, and a singular Gram matrix."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _basis(D):
    """D products of two atoms of w = [x (6); u (2)] from {1, w, sin w, cos w}, distinct functions."""
    atoms = [("one", 0)] + [("var", k) for k in range(8)] + [("sin", k) for k in range(8)]
    feats = [(0, 0)] + [(a, 0) for a in range(1, 17)] + [(a, b) for a in range(1, 9) for b in range(a, 9)] + \
        [(a, b) for a in range(9, 17) for b in range(a, 17)]
    return atoms, feats[:D]


def _lift(atoms, feats, W):
    fn = {"one": lambda v: np.ones(len(W)), "var": lambda v: W[:, v], "sin": lambda v: np.sin(W[:, v])}
    A = [fn[k](v) for k, v in atoms]
    return np.stack([A[p] * A[q] for p, q in feats], axis=1)


@pytest.mark.parametrize("D,T", [(1, 1), (15, 63), (16, 64), (17, 65), (31, 16384), (33, 16385), (48, 1000),
                                 (49, 40000), (63, 640), (64, 64), (64, 20000)])
def test_fit_and_lifted_fit_match_numpy(D, T):
    from paper_1906_02318_amd import mpmi

    rng = np.random.default_rng(1000 * D + T)
    X, U, Y = (rng.uniform(-2.0, 2.0, size=(T, k)) for k in (6, 2, 6))
    atoms, feats = _basis(D)
    sys = mpmi.custom_system(6, 2, atoms, feats, [], (-2.0, -2.0), (2.0, 2.0))
    P = _lift(atoms, feats, np.concatenate([X, U], axis=1))
    PY = _lift(atoms, feats, np.concatenate([Y, U], axis=1))
    s = np.sqrt(np.mean(P * P, axis=0))
    sv = np.linalg.svd(P / s, compute_uv=False)
    cond = sv[0] / sv[-1]
    ctx = mpmi.Context(0)
    d = [torch.tensor(v, device="cuda") for v in (X, U, Y)]
    for fit, target in ((mpmi.koopman_fit, Y), (mpmi.koopman_fit_lifted, PY)):
        if cond > 1e5:  # D = T: the normal equations hold no digits; the call must still end
            try:
                fit(ctx, sys, *d)
            except mpmi.MpmiError as e:
                assert e.status == mpmi.ESINGULAR
            continue
        K, c = fit(ctx, sys, *d)
        want = np.linalg.lstsq(P / s, target, rcond=None)[0]
        got = K.cpu().numpy() * s[:, None]
        # Normal equations: backward error of order D eps in the Gram matrix, amplified by cond^2.
        tol = 20 * D * np.finfo(np.float64).eps * cond ** 2 * np.linalg.norm(want)
        assert np.linalg.norm(got - want) <= max(tol, 1e-13)
        # 60 power steps from a fixed start bound the extreme eigenvalues from inside.
        assert 0.2 * cond <= c <= cond * (1 + 1e-9 + 20 * D * np.finfo(np.float64).eps * cond ** 2)


def test_dependent_features_are_reported_singular():
    from paper_1906_02318_amd import mpmi

    rng = np.random.default_rng(7)
    X, U, Y = (torch.tensor(rng.uniform(-1.0, 1.0, size=(500, k)), device="cuda") for k in (6, 2, 6))
    atoms, feats = _basis(40)
    sys = mpmi.custom_system(6, 2, atoms, feats + [feats[20]], [], (-2.0, -2.0), (2.0, 2.0))
    ctx = mpmi.Context(0)
    for fit in (mpmi.koopman_fit, mpmi.koopman_fit_lifted):
        with pytest.raises(mpmi.MpmiError) as e:
            fit(ctx, sys, X, U, Y)
        assert e.value.status == mpmi.ESINGULAR
