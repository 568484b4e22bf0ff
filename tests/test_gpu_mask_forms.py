"""Safety masks in both forms, four waves over the horizon in growing rounds
and one wave in chunks of four steps: first violations, least margins and the
near-boundary bits of a float32 scan step by step, at horizons around every
round's and chunk's end, and the same for a cloud as for its parts."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import synth
from paper_1906_02318_amd import mpmi
from tests import workloads as W

pytestmark = pytest.mark.gpu


def _bits(words, N):
    return np.unpackbits(words.cpu().numpy().view(np.uint8), bitorder="little")[:N].astype(bool)


# one candidate, a wave and a lane, ragged; both sides of the limit between the forms
_HORIZONS = [1, 3, 4, 5, 11, 12, 13, 28, 29, 60, 61, 92, 93, 255]
_SCANS = [(H, N, b) for N, b in ((1, [4]), (65, [0, 2, 4]), (300, [0, 1, 2, 3])) for H in _HORIZONS] + \
    [(H, N, [0, 2, 4]) for N in (98304, 98305) for H in (1, 3, 4, 5, 13)]


@pytest.mark.parametrize("H,N,boxed", _SCANS)
def test_against_a_scan(H, N, boxed):
    n = 4 if len(boxed) == 4 else 6  # with four components: every one constrained
    rng = np.random.default_rng(1000 * H + N)
    scale = 0.875 / max(2.0, np.sqrt(2.0 * np.log(max(2, H * len(boxed)))))  # verdicts on both sides
    traj = rng.normal(0.0, scale, size=(H, n, N)).astype(np.float32)
    for j in range(n):
        traj[:, j].flat[rng.integers(traj[:, j].size, size=3)] = [np.nan, np.inf, -np.inf][:3]
    eps = np.float32(0.03125)
    sys = mpmi.linear_system(n, 1, [(k, 1.0, 0.125) for k in boxed], [-1.0], [1.0])
    for b in range(len(boxed)):
        sys.eps32_box[b] = float(eps)
    ctx = mpmi.Context(0)
    model = mpmi.mpmi_model_pack(ctx, sys, torch.tensor(np.eye(n + 1, n), device="cuda"))
    dev = mpmi.new_traj(ctx, H, n, N)
    dev.copy_(torch.tensor(traj))
    each = np.float32(0.875) - np.abs(traj[:, boxed])
    want, low, near = np.full(N, H + 1), np.full(N, np.inf, dtype=np.float32), np.zeros(N, bool)
    for s in range(H):
        m, going = np.min(each[s], axis=0), want == H + 1
        near |= going & (np.abs(each[s]) < eps).any(axis=0)
        low = np.where(going, np.where(np.isnan(m), m, np.fmin(low, m)), low)
        want[going & ~(m > 0)] = s + 1
    fv, least, words = mpmi.safe_mask(ctx, model, dev, with_near=True)
    assert np.array_equal(fv.cpu().numpy(), want)
    assert np.array_equal(least.cpu().numpy(), low, equal_nan=True)
    assert np.array_equal(_bits(words, N), near)
    fv2, least2 = mpmi.safe_mask(ctx, model, dev)
    assert torch.equal(fv, fv2) and np.array_equal(least2.cpu().numpy(), low, equal_nan=True)


# a race car's three constrained components, and all six
@pytest.mark.parametrize("boxes", [[4], [2, 3, 4, 5]])
@pytest.mark.parametrize("H", [1, 5, 61])
def test_a_cloud_as_its_parts(boxes, H):
    N = 98304 + 97
    tr = W.rc_track()
    sys = mpmi._sys(mpmi.BASIS_RACE_CAR, 6, 2, [(k, 2.0, 0.0) for k in boxes], synth.RC_U_LO, synth.RC_U_HI,
                    track=W.track_dict(tr), eps32_box=[0.05] * len(boxes), eps32_track=1.0)
    ctx = mpmi.Context(0)
    model = mpmi.mpmi_model_pack(ctx, sys, torch.tensor(W.rc_model()[0], device="cuda"))
    g = torch.Generator(device="cuda").manual_seed(H)
    traj = mpmi.new_traj(ctx, H, 6, N)
    traj.copy_(0.3 * torch.randn((H, 6, N), generator=g, device="cuda"))
    phi = 6.2831853 * torch.rand((H, N), generator=g, device="cuda")
    rho = sum(float(a) * torch.sin(float(f) * phi + float(p)) for a, f, p in zip(tr.amp, tr.freq, tr.phase)) + tr.r0
    rho = rho + 0.7 * torch.randn((H, N), generator=g, device="cuda")
    traj[:, 0], traj[:, 1] = rho * torch.cos(phi), rho * torch.sin(phi)
    for j in range(6):
        at = torch.randint(0, N, (3,), generator=g, device="cuda")
        traj[H // 2, j, at] = torch.tensor([float("nan"), float("inf"), 0.0], device="cuda")
    fv, least, words = mpmi.safe_mask(ctx, model, traj, with_near=True)
    near = _bits(words, N)
    assert 0 < int((fv <= H).sum()) < N and 0 < near.sum() < N
    for a, b in ((0, 98304), (32, 96), (128, N), (98304, N)):
        part = mpmi.safe_mask(ctx, model, traj[:, :, a:b], with_near=True)
        assert torch.equal(part[0], fv[a:b])
        assert torch.equal(part[1].view(torch.int32), least[a:b].view(torch.int32))
        assert np.array_equal(_bits(part[2], b - a), near[a:b])
