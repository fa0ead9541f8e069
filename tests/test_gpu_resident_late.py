"""Stop decisions of the resident solve that fall a sweep late, against the launch-per-sweep path.

While no stop is in sight the decision on round t - 2 falls at the end of sweep t, and a sweep too
many is taken back.  Whether a stop is in sight is judged by the last rate of decay, so the cases
here are those where that judgement fails: a residual that collapses when the messages of a tree
have met, one that rises beyond the divergence limit, tolerances around a round's own residual,
and caps on the sweeps around the stop.  The two paths perform the same operations: x, the
variances and the sweep counts are equal bit for bit, and the residual, summed in another order,
to 1e-12.
"""
import numpy as np
import pytest
import torch

import paper_0811_2518_amd as g
import workloads

pytestmark = pytest.mark.gpu
DEV = "cuda"


def dev(v):
    return torch.from_numpy(np.ascontiguousarray(v)).to(DEV)


CASES = {
    "tree": lambda: workloads.random_tree(9777, 81),           # exact once every message has arrived
    "grid_97x61": lambda: workloads.grid2d_problem(97, 61, 2),
    "er_60000": lambda: workloads.er_problem(60000, 8, 78),    # chains, 512 lanes
}


def both(p, b, tol, M, val=None, **kw):
    out = []
    for multi in (False, True):
        s = g.Solver(p.row_ptr, p.col, p.val if val is None else val, device=DEV, layout="compact",
                     reuse_precision=False, multi_launch=multi, **kw)
        x, i, v = s.solve(b, tol=tol, max_iter=M, var=True, check=False)
        out.append((x, i, v))
        s.close()
    (x1, i1, v1), (x2, i2, v2) = out
    assert (i1["sweeps"], i1["converged"], i1["status"]) == (i2["sweeps"], i2["converged"], i2["status"]), (tol, M)
    assert i1["rel_residual"] == pytest.approx(i2["rel_residual"], rel=1e-12, abs=1e-300)
    if i1["status"] >= 0:  # an error leaves x undefined
        assert torch.equal(x1, x2) and torch.equal(v1, v2), (tol, M)
    return i1


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("check_every", [1, 3])
def test_stops_fall_on_the_same_round(name, check_every):
    p = CASES[name]()
    b = dev(p.b)
    last = both(p, b, 1e-10, 500, check_every=check_every)
    T = last["sweeps"]
    assert last["converged"] == 1
    for M in (T - 1, T, T + 1, T + 2):
        both(p, b, 1e-10, M, check_every=check_every)
    for tol in (0.9, 0.05, 1e-3, 1e-13):
        both(p, b, tol, 500, check_every=check_every)


def test_a_diverging_solve_ends_on_the_same_round():
    p = workloads.grid2d_problem(97, 61, 2)
    val = p.val.copy()
    rows = np.repeat(np.arange(p.n), np.diff(p.row_ptr))
    val[rows == p.col] *= 0.45  # far from diagonal dominance
    for M in (20, 500):
        assert both(p, dev(p.b), 1e-10, M, val=val)["converged"] == 0


def test_frozen_precisions():
    p = workloads.er_problem(60000, 8, 78)
    rng = np.random.default_rng(5)
    sol = [g.Solver(p.row_ptr, p.col, p.val, device=DEV, layout="compact", multi_launch=m) for m in (False, True)]
    for k in range(3):
        b = dev(rng.standard_normal(p.n))
        (x1, i1), (x2, i2) = [s.solve(b, tol=1e-10, max_iter=500) for s in sol]
        assert i1["sweeps"] == i2["sweeps"] and torch.equal(x1, x2), k
