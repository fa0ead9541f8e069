"""Solves that get no place on the chip for their resident launch.

The roll call is made to fail from the host (a limit of zero), as it does when other work holds
the chip, and the solve takes the launch-per-sweep path.  Whether a chip is busy must not show in
a result: x, the variances, the sweeps and the outer steps are those of the resident launch bit for
bit, and later solves of the handle are untouched by the failed launch.
"""
import threading
import time

import numpy as np
import pytest
import torch

import paper_0811_2518_amd as g
import workloads

from _aids import ABORTED, LARGEST_TEAM, ROLL_LIMIT, get_aid, set_aid

pytestmark = pytest.mark.gpu
DEV = "cuda"


def dev(v):
    return torch.from_numpy(np.ascontiguousarray(v)).to(DEV)


PROBS = {
    "grid_97x61": lambda: workloads.grid2d_problem(97, 61, 2),
    "grid_181x173": lambda: workloads.grid2d_problem(181, 173, 3),
    "er_30011": lambda: workloads.er_problem(30011, 8, 77),
    "tree": lambda: workloads.random_tree(9777, 81),
    "btb_3000": lambda: workloads.config5(n=3000, rows=6000),
}
MODES = {
    "plain": ("grid_181x173", {"reuse_precision": False}),
    "reuse": ("er_30011", {}),
    "serial": ("grid_97x61", {"layout": "serial"}),
    "fp32": ("er_30011", {"precision": "fp32", "reuse_precision": False}),
    # the residual collapses when the messages have met, which no rate of decay predicts
    "fp32_tree": ("tree", {"precision": "fp32", "reuse_precision": False}),
    "fp32_reuse": ("grid_181x173", {"precision": "fp32"}),
    "fp32_serial": ("grid_97x61", {"precision": "fp32", "layout": "serial"}),
    "loaded_fp32": ("btb_3000", {"precision": "fp32", "gamma": -1.0, "inner_tol": 1e-2, "max_outer": 5000}),
    "loaded_fp64": ("btb_3000", {"gamma": -1.0, "inner_tol": 1e-2, "max_outer": 5000, "reuse_precision": False}),
    "single_fp64": ("btb_3000", {"gamma": -1.0, "inner_tol": 1e-3, "single_loop": True}),
    "single_fp32": ("btb_3000", {"gamma": -1.0, "inner_tol": 1e-3, "single_loop": True, "precision": "fp32",
                                 "max_outer": 5000}),
}


@pytest.mark.parametrize("mode", sorted(MODES))
def test_results_do_not_depend_on_the_load(mode):
    name, kw = MODES[mode]
    p = PROBS[name]()
    rng = np.random.default_rng(9)
    bs = [dev(p.b), dev(rng.standard_normal(p.n)), dev(rng.standard_normal(p.n))]
    var = "gamma" not in kw and kw.get("precision") != "fp32"

    def run(limits):
        s = g.Solver(p.row_ptr, p.col, p.val, device=DEV, **kw)
        out = []
        for b, limit in zip(bs, limits):
            set_aid(s, ROLL_LIMIT, limit)
            before = get_aid(s, ABORTED)
            got = s.solve(b, tol=1e-9, max_iter=200000, var=var)
            assert (get_aid(s, ABORTED) > before) == (limit == 1)
            out.append(got)
        s.close()
        return out

    want = run((0, 0, 0))
    for limits in ((1, 1, 1), (1, 0, 1), (0, 1, 0)):
        for got, ref in zip(run(limits), want):
            assert torch.equal(got[0], ref[0]), limits
            assert all(got[1][k] == ref[1][k] for k in ("sweeps", "outer_iters", "converged", "status")), limits
            assert got[1]["rel_residual"] == pytest.approx(ref[1]["rel_residual"], rel=1e-12), limits
            if var:
                assert torch.equal(got[2], ref[2]), limits


BATCHES = {
    "one_er": lambda: ([workloads.er_problem(40001, 8, 1, ratio=1.1)], [1]),
    "one_grid3d": lambda: ([workloads.grid3d_problem(24, 2)], [8]),
    "mixed": lambda: ([workloads.grid2d_problem(121, 101, 6, ratio=1.1), workloads.er_problem(9001, 12, 7),
                       workloads.grid3d_problem(13, 8)] + [workloads.grid2d_problem(9 + q % 5, 8, 20 + q) for q in range(40)],
                      [3, 7, 1] + [1 + q % 5 for q in range(40)]),
}


@pytest.mark.parametrize("layout", ["auto", "serial"])
@pytest.mark.parametrize("name", sorted(BATCHES))
def test_batches_do_not_depend_on_the_load(name, layout):
    probs, ks = BATCHES[name]()
    bt = workloads.batch_of(probs, ks, seed=54)
    s = g.BatchedSolver(bt.sys_row_off, bt.row_ptr, bt.col, bt.val, device=DEV, layout=layout)
    rng = np.random.default_rng(11)
    B = [dev(bt.B)] + [dev(rng.standard_normal(len(bt.B))) for _ in range(3)]

    def run(limit):
        out = []
        for b in B:
            set_aid(s, ROLL_LIMIT, limit)
            X, infos, st = s.solve(bt.nrhs, bt.rhs_off, b, tol=1e-10, max_iter=20000)
            assert st == 0 and (get_aid(s, LARGEST_TEAM) > 1) == (limit == 0)
            out.append((X, [(i["sweeps"], i["outer_iters"], i["rel_residual"]) for i in infos]))
        return out

    want = run(0)
    for limit in (1, 0):
        for (X, infos), (Xw, iw) in zip(run(limit), want):
            assert torch.equal(X, Xw) and infos == iw, limit


def test_a_chip_out_of_reach_is_tried_ever_more_rarely():
    """Each try spins for the limit of a roll call, so failures in a row are tried 1, 2, 4, ... calls
    apart; the calls between give the same result, and a success starts anew."""
    p = PROBS["grid_97x61"]()
    bt = workloads.batch_of([workloads.er_problem(30001, 8, 1, ratio=1.1)], [1], seed=55)
    s = g.Solver(p.row_ptr, p.col, p.val, device=DEV, reuse_precision=False)
    sb = g.BatchedSolver(bt.sys_row_off, bt.row_ptr, bt.col, bt.val, device=DEV)
    b, B = dev(p.b), dev(bt.B)

    def one():
        return s.solve(b, tol=1e-10, max_iter=2000)[0]

    def batch():
        return sb.solve(bt.nrhs, bt.rhs_off, B, tol=1e-10, max_iter=20000)[0]

    for h, solve in ((s, one), (sb, batch)):
        want = solve()
        assert get_aid(h, ABORTED) == 0
        set_aid(h, ROLL_LIMIT, 1)
        tried = []
        for _ in range(22):
            before = get_aid(h, ABORTED)
            assert torch.equal(solve(), want)
            tried.append(get_aid(h, ABORTED) - before)
        assert [k for k, v in enumerate(tried) if v] == [0, 2, 5, 10, 19]
        set_aid(h, ROLL_LIMIT, 0)
        n = get_aid(h, ABORTED)
        assert torch.equal(solve(), want) and get_aid(h, ABORTED) == n


def test_a_thread_whose_stream_is_busy_keeps_nobody_waiting():
    """A thread's solve stands behind 0.6 s of other work of its stream (one lane, so it takes no
    room on the chip).  A batch and a solve of another thread finish meanwhile."""
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda._sleep(1000)
    start.record()
    torch.cuda._sleep(10_000_000)
    end.record()
    end.synchronize()
    cycles = int(10_000_000 * 600.0 / start.elapsed_time(end))
    p = PROBS["grid_181x173"]()
    bt = workloads.batch_of([workloads.er_problem(30001, 8, 1, ratio=1.1)], [1], seed=56)
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    a = g.Solver(p.row_ptr, p.col, p.val, device=DEV, reuse_precision=False, stream=sa)
    b = g.Solver(p.row_ptr, p.col, p.val, device=DEV, reuse_precision=False, stream=sb)
    bb = g.BatchedSolver(bt.sys_row_off, bt.row_ptr, bt.col, bt.val, device=DEV, stream=sb)
    rhs, B = dev(p.b), dev(bt.B)
    xa, xb, X = torch.empty_like(rhs), torch.empty_like(rhs), torch.empty_like(B)
    a.solve(rhs, tol=1e-10, max_iter=2000, x=xa)
    b.solve(rhs, tol=1e-10, max_iter=2000, x=xb)
    bb.solve(bt.nrhs, bt.rhs_off, B, tol=1e-10, max_iter=20000, X=X)
    torch.cuda.synchronize()
    errors, done, queued = [], threading.Event(), threading.Event()

    def first(wait):
        try:
            with torch.cuda.stream(sa):
                if wait:
                    torch.cuda._sleep(cycles)
                queued.set()
                a.solve(rhs, tol=1e-10, max_iter=2000, x=xa)
        except Exception as e:  # reported by the main thread
            errors.append(e)
        done.set()

    t = threading.Thread(target=first, args=(False,))  # now two threads have used the chip
    t.start()
    t.join()
    done.clear()
    queued.clear()
    t = threading.Thread(target=first, args=(True,))
    t.start()
    queued.wait()
    time.sleep(0.02)  # inside its solve by now
    with torch.cuda.stream(sb):
        b.solve(rhs, tol=1e-10, max_iter=2000, x=xb)
        bb.solve(bt.nrhs, bt.rhs_off, B, tol=1e-10, max_iter=20000, X=X)
    early = not done.is_set()
    t.join()
    assert not errors, errors
    assert early and torch.equal(xa, xb)
