"""Batched items that a team of workgroups runs.

An item that would outlast an even share of the batch is split over 2 to 64
workgroups.  The cases cover one large system alone (the largest team), large
systems among small ones (several team sizes and single workgroups in one
launch), systems at the edges of a team (one 64-row slice per wave and one row
more), and both schedules.  Every solution is held to its relative residual in
FP64 and to a conjugate-gradient reference.
"""
import numpy as np
import pytest
import scipy.sparse.linalg as spla
import torch

import paper_0811_2518_amd as g
import workloads
from paper_0811_2518_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda"
TOL = 1e-10

CASES = {
    "one_large": lambda: ([workloads.er_problem(40000, 8, 1, ratio=1.1)], [1]),
    "one_large_8_rhs": lambda: ([workloads.grid3d_problem(24, 2)], [8]),
    "slice_edges": lambda: ([workloads.grid2d_problem(32, 32, 3, ratio=1.2), workloads.grid2d_problem(41, 25, 4, ratio=1.2),
                             workloads.er_problem(1023, 6, 5)], [1, 1, 2]),
    "mixed": lambda: ([workloads.grid2d_problem(120, 101, 6, ratio=1.1), workloads.er_problem(9001, 12, 7),
                       workloads.grid3d_problem(13, 8)] + [workloads.grid2d_problem(9 + q % 5, 8, 20 + q) for q in range(40)],
                      [3, 7, 1] + [1 + q % 5 for q in range(40)]),
    "hub": lambda: ([workloads.powerlaw_problem(20000, 8, 9, beta=2.1)], [2]),
}


@pytest.mark.parametrize("layout", ["auto", "serial"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_team_solutions(name, layout):
    probs, ks = CASES[name]()
    bt = workloads.batch_of(probs, ks, seed=51)
    s = g.BatchedSolver(bt.sys_row_off, bt.row_ptr, bt.col, bt.val, device=DEV, layout=layout)
    B = torch.from_numpy(bt.B).to(DEV)
    X, infos, st = s.solve(bt.nrhs, bt.rhs_off, B, tol=TOL, max_iter=20000)
    assert st == binding.OK
    Xh = X.cpu().numpy()
    for q, info in enumerate(infos):
        assert info["converged"] == 1 and info["rel_residual"] <= TOL, (q, info)
        p = bt.system(q)
        k = p.b.shape[1]
        A = p.scipy()
        xs = Xh[bt.rhs_off[q]:bt.rhs_off[q + 1]].reshape(p.n, k)
        for j in range(k):
            b = p.b[:, j]
            assert np.linalg.norm(b - A @ xs[:, j]) <= 1.05 * TOL * np.linalg.norm(b), (q, j)
            ref, ok = spla.cg(A, b, rtol=1e-13, atol=0.0, maxiter=20000)
            # a residual of 1e-10 through a condition number of at most 41
            assert ok == 0 and np.linalg.norm(xs[:, j] - ref) <= 1e-8 * np.linalg.norm(ref), (q, j)
    # new buffers and another right-hand side on the same work list, then the first again: same bits
    B2 = torch.from_numpy(np.random.default_rng(3).standard_normal(len(bt.B))).to(DEV)
    X2, infos2, st2 = s.solve(bt.nrhs, bt.rhs_off, B2, tol=TOL, max_iter=20000)
    X3, infos3, st3 = s.solve(bt.nrhs, bt.rhs_off, B.clone(), tol=TOL, max_iter=20000)
    assert st2 == st3 == binding.OK and not torch.equal(X2, X3)
    assert torch.equal(X, X3) and [i["sweeps"] for i in infos] == [i["sweeps"] for i in infos3]
    # another grouping of the right-hand sides plans anew
    if sum(ks) > len(ks):
        ones = np.ones(len(ks), np.int32)
        off = np.concatenate([[0], np.cumsum([p.n for p in probs])]).astype(np.int64)
        b1 = torch.ones(int(off[-1]), dtype=torch.float64, device=DEV)
        x1, _, st1 = s.solve(ones, off, b1, tol=TOL, max_iter=20000)
        assert st1 == binding.OK
        for q, p in enumerate(probs):
            r = np.ones(p.n) - p.scipy() @ x1[off[q]:off[q + 1]].cpu().numpy()
            assert np.linalg.norm(r) <= 1.05 * TOL * np.sqrt(p.n), q


def test_teams_beside_other_work():
    """Two handles on streams of their own while products fill the chip: each launch either gets
    its workgroups in time or runs every item in a single workgroup, with the same solutions."""
    probs, ks = CASES["mixed"]()
    bt = workloads.batch_of(probs, ks, seed=52)
    B = torch.from_numpy(bt.B).to(DEV)
    s0 = g.BatchedSolver(bt.sys_row_off, bt.row_ptr, bt.col, bt.val, device=DEV)
    want = s0.solve(bt.nrhs, bt.rhs_off, B, tol=TOL, max_iter=20000)[0]
    torch.cuda.synchronize()
    import threading
    got, errors = [], []

    def work():
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                s = g.BatchedSolver(bt.sys_row_off, bt.row_ptr, bt.col, bt.val, device=DEV)
                for _ in range(4):
                    got.append(s.solve(bt.nrhs, bt.rhs_off, B, tol=TOL, max_iter=20000)[0])
        except Exception as e:  # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work) for _ in range(2)]
    for t in threads:
        t.start()
    a = torch.randn(8192, 8192, device=DEV)
    for _ in range(20):
        a = (a @ a) * 1e-3
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for x in got:
        # the means of a round do not depend on the split; only sums of squares do, in their last bits
        assert float((x - want).norm() / want.norm()) <= 1e-9
