"""Two-lane builds on reduced workspaces and in a captured graph: the same bits as on one
stream.
"""
import numpy as np
import pytest

import _gpu as G
from test_slice_steps_gpu import _inputs, _set

pytestmark = pytest.mark.gpu


# 161 and 97 beams; chunks of 5, 41 and all but one of them (state of a beam: 1.0 / 1.3 MiB)
@pytest.mark.parametrize("n,f,H", [(512, 4, 4), (576, 6, 4)])
def test_two_lanes_on_reduced_workspaces(n, f, H):
    d = _inputs(n, H, 21)
    amax = _set(n, f, 20.0)
    plan = G.make_plan(d)
    B = plan.beam_count(f, amax)
    wave = n * (n // 2) * 8
    assert 4.0 * B * H * wave >= 2 ** 30  # two lanes
    plan.profile(True)  # one lane
    one = G.build_smatrix(plan, f, amax).cpu().numpy().view(np.uint64)
    plan.profile(False)
    least = plan.build_workspace_bytes(f, amax)[1]
    for waves in (1, 2, 3, 5, 41, B - 1):
        S = G.build_smatrix(plan, f, amax, ws_bytes=least + (waves - 1) * wave)
        assert np.array_equal(S.cpu().numpy().view(np.uint64), one), waves


def test_two_lane_build_in_a_graph():
    """Captured on a plan that has not built before (its second stream is created inside the
    capture) and on one that has; replays with eager work between them."""
    import torch
    n, f, H = 512, 4, 4
    d = _inputs(n, H, 22)
    amax = _set(n, f, 20.0)
    for cold in (True, False):
        plan, other = G.make_plan(d), G.make_plan(d)
        B = plan.beam_count(f, amax)
        ref = G.build_smatrix(other, f, amax).clone()
        if not cold:
            G.build_smatrix(plan, f, amax)
        S = torch.zeros((B, n // 2, n // 2), dtype=torch.complex64, device=G.device())
        ws = G.workspace(plan.build_workspace_bytes(f, amax)[0])
        G.say(f"capture a two-lane build, cold={cold}")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            plan.build_smatrix(f, amax, S, ws, stream=torch.cuda.current_stream())
        for _ in range(3):
            S.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(torch.view_as_real(S), torch.view_as_real(ref))
            assert torch.equal(torch.view_as_real(G.build_smatrix(other, f, amax)),
                               torch.view_as_real(ref))
        del graph
