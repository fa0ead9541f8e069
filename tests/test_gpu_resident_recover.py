"""The resident solve after a launch that did not run or whose workgroups gave up.

A launch clears the barrier counters that the next one uses.  One that was recorded into a stream
capture (a solve waits for its result, so the call ends in an error) or refused never runs, and
what it should have cleared must not let the next solve's barriers through.
"""
import ctypes

import numpy as np
import pytest
import torch

import paper_0811_2518_amd as g
import workloads
from paper_0811_2518_amd import binding

from _aids import WAIT_LIMIT, set_aid

pytestmark = pytest.mark.gpu
DEV = "cuda"
THREAD_LOCAL = 1  # hipStreamCaptureModeThreadLocal


def dev(v):
    return torch.from_numpy(np.ascontiguousarray(v)).to(DEV)


@pytest.mark.parametrize("layout", ["auto", "serial"])
@pytest.mark.parametrize("name", ["grid_97x61", "grid_181x173"])  # one counter, counters in groups
@pytest.mark.parametrize("before", [0, 1, 2])
def test_solve_after_a_refused_capture(name, layout, before):
    px, py = (97, 61) if name == "grid_97x61" else (181, 173)
    p = workloads.grid2d_problem(px, py, 2)
    hip = binding.lib()  # finds the runtime that the library itself uses
    st = torch.cuda.Stream()
    sh = ctypes.c_void_p(st.cuda_stream)

    def end_capture():
        graph = ctypes.c_void_p()
        hip.hipStreamEndCapture(sh, ctypes.byref(graph))
        if graph.value:
            hip.hipGraphDestroy(graph)
        hip.hipGetLastError()

    with torch.cuda.stream(st):
        s = g.Solver(p.row_ptr, p.col, p.val, device=DEV, layout=layout, reuse_precision=False, stream=st)
        multi = g.Solver(p.row_ptr, p.col, p.val, device=DEV, layout="compact" if layout == "auto" else layout,
                         reuse_precision=False, multi_launch=True, stream=st)
        b = dev(p.b)
        x, out = torch.empty_like(b), torch.empty_like(b)
        want, wi = multi.solve(b, tol=1e-10, max_iter=2000)
        for _ in range(before):
            assert torch.equal(s.solve(b, tol=1e-10, max_iter=2000)[0], want)
        st.synchronize()
        for _ in range(2):  # two in a row: either control block may be the one left behind
            assert hip.hipStreamBeginCapture(sh, THREAD_LOCAL) == 0
            info = s.solve(b, tol=1e-10, max_iter=2000, x=out, check=False)[1]
            end_capture()
            assert info["status"] == binding.E_HIP
            # the stream stays marked as invalidated until its next capture, here an empty one
            assert hip.hipStreamBeginCapture(sh, THREAD_LOCAL) == 0
            end_capture()
            for _ in range(3):
                x.zero_()
                _, i = s.solve(b, tol=1e-10, max_iter=2000, x=x)
                assert torch.equal(x, want) and i["sweeps"] == wi["sweeps"]
        st.synchronize()


@pytest.mark.parametrize("kw", [{}, {"layout": "serial"}, {"precision": "fp32"}], ids=["plain", "serial", "fp32"])
@pytest.mark.parametrize("name", ["grid_97x61", "grid_181x173"])
def test_a_workgroup_that_stops_waiting_is_reported(name, kw):
    """Waits cut short by a tiny limit: whichever workgroup gives up, the call ends in an error or
    with the very bits of a full solve, and the handle solves again afterwards."""
    px, py = (97, 61) if name == "grid_97x61" else (181, 173)
    p = workloads.grid2d_problem(px, py, 2)
    s = g.Solver(p.row_ptr, p.col, p.val, device=DEV, **kw)
    b = dev(p.b)
    want = [s.solve(b, tol=1e-10, max_iter=2000)[0] for _ in range(2)]
    s.close()
    s = g.Solver(p.row_ptr, p.col, p.val, device=DEV, **kw)
    seen = set()
    for ticks in (0, 20, 50, 100, 150, 200, 300, 500, 1000, 10000):
        for _ in range(3):
            set_aid(s, WAIT_LIMIT, ticks + 1)
            x, info = s.solve(b, tol=1e-10, max_iter=2000, check=False)
            seen.add(info["status"])
            assert info["status"] in (binding.OK, binding.E_HIP), info
            if info["status"] == binding.OK:  # plain reuse: the first solve, or one on its frozen precisions
                assert any(torch.equal(x, w) for w in want), ticks
            set_aid(s, WAIT_LIMIT, 0)
            x, info = s.solve(b, tol=1e-10, max_iter=2000)
            assert any(torch.equal(x, w) for w in want), ticks
    assert binding.E_HIP in seen  # no barrier ends within the first look at the clock
