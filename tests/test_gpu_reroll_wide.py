"""The FP64 re-roll of a basis of 64 features over lists on both sides of the
limit above which smaller bases take one candidate per lane: bands so wide that
every candidate is kept, against a float64 prediction here.  The two add the
same terms in other orders and so agree to some 1e-13; that no margin is closer
to zero than 1e-11 is asserted."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_1906_02318_amd import mpmi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [32766, 32767, 32768, 40001])
def test_wide_basis_first_violations_are_a_float64_predictions(N):
    rng = np.random.default_rng(N)
    n, m, D, H, S = 6, 2, 64, 12, 2
    atoms = [("one", 0)] + [(k, v) for k in ("var", "sin", "cos") for v in range(n + m)]
    feats = [(1 + k, 0) for k in range(n + m)]
    while len(feats) < D:
        feats.append((int(rng.integers(len(atoms))), int(rng.integers(len(atoms)))))
    sys = mpmi.custom_system(n, m, atoms, feats, [(0, 0.9, 0.0), (3, 1.1, 0.0)], [-1.0] * m, [1.0] * m,
                             eps32_box=[1e30] * 2)
    K = 0.03 * rng.standard_normal((D, n))
    K[np.arange(n), np.arange(n)] += 0.97
    ctx = mpmi.Context(0)
    model = mpmi.mpmi_model_pack(ctx, sys, torch.tensor(K, device="cuda"))
    x = (0.4 * rng.standard_normal(n)).astype(np.float32)
    cand = rng.uniform(-1.0, 1.0, size=(S, m, N + 1)).astype(np.float32)  # the first: the user's input, held
    cand[1:, :, 0] = cand[0, :, 0]
    fv = torch.zeros(N + 1, dtype=torch.int16, device="cuda")
    rec = mpmi.mpmi_tick(ctx, model, mpmi.tick_desc(N, H, gen=mpmi.GEN_EXPLICIT, n_seg=S,
                                                    precision=mpmi.PREC_FP32_RECHECK64),
                         torch.tensor(x, device="cuda"), torch.tensor(cand[0, :, 0], device="cuda"),
                         cand=torch.tensor(cand[:, :, 1:], device="cuda").contiguous(), first_violation=fv)
    assert mpmi.decode_selection(rec)["n_recheck"] == N + 1
    X = np.repeat(x.astype(np.float64)[:, None], N + 1, axis=1)
    want, least = np.full(N + 1, H + 1), np.inf
    for s in range(1, H + 1):
        w = np.concatenate([X, cand[((s - 1) * S) // H].astype(np.float64)])
        at = [{"one": np.ones_like, "var": lambda v: v, "sin": np.sin, "cos": np.cos}[k](w[v]) for k, v in atoms]
        X = K.T @ np.stack([at[a] * at[b] for a, b in feats])
        margin = np.minimum(0.9 - np.abs(X[0]), 1.1 - np.abs(X[3]))
        going = want == H + 1
        least = min(least, np.min(np.abs(margin[going]), initial=np.inf))
        want[going & ~(margin > 0)] = s
    assert 0 < (want <= H).sum() <= N and least > 1e-11
    assert np.array_equal(fv.cpu().numpy(), want)
