"""Teams of a batched solve whose members sit on one XCD, and on different ones.

Members exchange their data past the caches of an XCD, so where they sit must not change a bit:
neither the frozen coefficients of the precision phase nor the solutions.  The systems' colour
classes are not multiples of a team's waves, so that a pass that dealt its slices otherwise than
the pass before it would read another workgroup's plain stores.
"""
import pytest
import torch

import paper_0811_2518_amd as g
import workloads
from paper_0811_2518_amd import binding

from _aids import SPREAD_TEAMS, set_aid

pytestmark = pytest.mark.gpu
DEV = "cuda"

CASES = {
    "one_er": lambda: ([workloads.er_problem(40001, 8, 1, ratio=1.1)], [1]),
    "one_grid3d": lambda: ([workloads.grid3d_problem(23, 2)], [5]),
    "mixed": lambda: ([workloads.grid2d_problem(121, 101, 6, ratio=1.1), workloads.er_problem(9001, 12, 7),
                       workloads.grid3d_problem(13, 8)] + [workloads.grid2d_problem(9 + q % 5, 8, 20 + q) for q in range(40)],
                      [3, 7, 1] + [1 + q % 5 for q in range(40)]),
}


@pytest.mark.parametrize("layout", ["auto", "serial"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_placement_changes_no_bit(name, layout):
    probs, ks = CASES[name]()
    bt = workloads.batch_of(probs, ks, seed=53)
    B = torch.from_numpy(bt.B).to(DEV)
    got = []
    for spread in (0, 1, 1, 0):
        s = g.BatchedSolver(bt.sys_row_off, bt.row_ptr, bt.col, bt.val, device=DEV, layout=layout)
        set_aid(s, SPREAD_TEAMS, spread)
        X, infos, st = s.solve(bt.nrhs, bt.rhs_off, B, tol=1e-10, max_iter=20000)
        assert st == binding.OK
        prof = s.profile()
        got.append((X, [(i["sweeps"], i["outer_iters"], i["rel_residual"]) for i in infos], prof["precision_sweeps"]))
        s.close()
    for X, infos, psweeps in got[1:]:
        assert torch.equal(X, got[0][0]) and infos == got[0][1] and psweeps == got[0][2]
