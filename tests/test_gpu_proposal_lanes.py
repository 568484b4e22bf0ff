"""A learned tick's launches: lanes_per_cand 1 runs one lane per candidate, 0
leaves the choice to the library, which spreads 2,048 proposals over eight
lanes and a fallback of 4,096 points too.  Read from the launch sizes of the
captured calls; nothing is launched for it."""
from __future__ import annotations

import ctypes

import pytest
import torch

import synth
from paper_1906_02318_amd import mpmi
from paper_1906_02318_amd.proposal import ASSET, LearnedTicker, ProposalNet
from tests import workloads as W

pytestmark = pytest.mark.gpu


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint), ("y", ctypes.c_uint), ("z", ctypes.c_uint)]


class _KernelParams(ctypes.Structure):  # hipKernelNodeParams
    _fields_ = [("block", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", _Dim3),
                ("args", ctypes.c_void_p), ("lds", ctypes.c_uint)]


def _launches(call):
    """(workgroups, threads per workgroup) of every kernel the call launches."""
    hip, stream = mpmi.library(), torch.cuda.Stream()
    graph, n = ctypes.c_void_p(), ctypes.c_size_t()
    with torch.cuda.stream(stream):
        s = ctypes.c_void_p(stream.cuda_stream)
        assert hip.hipStreamBeginCapture(s, 2) == 0  # relaxed
        try:
            call()
        finally:
            assert hip.hipStreamEndCapture(s, ctypes.byref(graph)) == 0
    try:
        assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
        nodes = (ctypes.c_void_p * n.value)()
        assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
        out = []
        for node in nodes:
            p = _KernelParams()
            assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
            out.append((p.grid.x, p.block.x))
        return out
    finally:
        assert hip.hipGraphDestroy(graph) == 0


@pytest.mark.parametrize("lanes,spread", [(None, 8), (0, 8), (1, 1), (2, 2), (4, 4)])
def test_the_launch_has_the_lanes_that_were_asked_for(lanes, spread):
    ctx = mpmi.Context(0)
    model = mpmi.mpmi_model_pack(ctx, mpmi.race_car_system(W.track_dict(W.rc_track())),
                                 torch.tensor(W.rc_model()[0], device="cuda"))
    kw = {} if lanes is None else dict(lanes_per_cand=lanes)
    ticker = LearnedTicker(ctx, model, ProposalNet.load(ctx, ASSET), proposals=2047, fallback_grid=(63, 65), **kw)
    x = torch.tensor(synth.race_car_states(1, W.rc_track(), seed=4)[0], dtype=torch.float32, device="cuda")
    u = torch.zeros(2, dtype=torch.float32, device="cuda")
    out = torch.zeros(mpmi.SELECTION_BYTES, dtype=torch.uint8, device="cuda")
    ticker.tick(x, u, tick=0, out=out)
    torch.cuda.synchronize()
    # network row with the proposals' draws, the tick over 2,048 candidates, the fallback over 4,096
    want = [(8, 1024), (8 * spread, 256), (16 * 8, 256)]
    assert sorted(_launches(lambda: ticker.tick(x, u, tick=1, out=out))) == sorted(want)
    ticker.fallback.lanes_per_cand = 1
    want[2] = (16, 256)
    assert sorted(_launches(lambda: ticker.tick(x, u, tick=1, out=out))) == sorted(want)
