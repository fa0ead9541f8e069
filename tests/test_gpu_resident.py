"""The resident solve of mid-sized systems against the launch-per-sweep path.

Compact solves that fit on the chip run every sweep, check, outer step and stop
decision in one launch of resident workgroups.  It performs the operations of
the launch-per-sweep path in the same order, so x, the variances, the messages,
the gradients and the sweep counts must agree bit for bit; the reported
residual is summed in another order (relative 1e-12).  The sizes straddle the
edges of the plan: one workgroup and several, rows of one lane and chains of
lanes, one counter and counters in groups, each workgroup size.
"""
import threading

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
    "grid_33x32": lambda: workloads.grid2d_problem(33, 32, 1),       # just beyond one workgroup
    "grid_97x61": lambda: workloads.grid2d_problem(97, 61, 2),       # one counter (24 workgroups)
    "grid_181x173": lambda: workloads.grid2d_problem(181, 173, 3),   # counters in groups
    "grid3d_11": lambda: workloads.grid3d_problem(11, 4),            # 6 slots a lane
    "grid3d_45": lambda: workloads.grid3d_problem(45, 5),            # 512 lanes
    "grid3d_64": lambda: workloads.grid3d_problem(64, 6),            # 1024 lanes, every CU
    "er_3001": lambda: workloads.er_problem(3001, 8, 77),            # chains of lanes, XCD parts
    "er_60000": lambda: workloads.er_problem(60000, 8, 78),          # chains, 512 lanes
    "er_isolated": lambda: workloads.er_problem(9000, 3, 82, ratio=1.3),
    "star_96": lambda: workloads.star_problem(96, 83),               # the longest chain: 16 lanes
    "star_97": lambda: workloads.star_problem(97, 84),               # one slot too many: launch per sweep
    "tree": lambda: workloads.random_tree(4777, 80),
}


def pair(p, **kw):
    one = g.Solver(p.row_ptr, p.col, p.val, device=DEV, **kw)
    multi = g.Solver(p.row_ptr, p.col, p.val, device=DEV, layout="compact", multi_launch=True, **kw)
    return one, multi


def same_info(i1, i2):
    for k in ("sweeps", "converged", "status"):
        assert i1[k] == i2[k], (k, i1, i2)
    assert i1["rel_residual"] == pytest.approx(i2["rel_residual"], rel=1e-12, abs=1e-300)


@pytest.mark.parametrize("name", sorted(CASES))
def test_fixed_rounds_bitwise(name):
    p = CASES[name]()
    one, multi = pair(p)
    assert one.props()["layout"] == 3
    b = dev(p.b)
    for T in (0, 1, 2, 3, 8):
        x1, i1, v1 = one.solve(b, tol=0, max_iter=T, var=True)
        x2, i2, v2 = multi.solve(b, tol=0, max_iter=T, var=True)
        assert torch.equal(x1, x2) and torch.equal(v1, v2), (name, T)
        same_info(i1, i2)
        for m1, m2 in zip(one.messages(), multi.messages()):
            assert torch.equal(m1, m2), (name, T)


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("check_every", [1, 3])
def test_converged_reuse_and_adjoint_bitwise(name, check_every):
    p = CASES[name]()
    rng = np.random.default_rng(5)
    b, b2 = dev(p.b), dev(rng.standard_normal(p.n))
    for reuse in (False, True):
        one, multi = pair(p, reuse_precision=reuse, check_every=check_every)
        for bv in (b, b2):  # with reuse, the second solve runs on frozen precisions
            x1, i1, v1 = one.solve(bv, tol=1e-10, max_iter=5000, var=True)
            x2, i2, v2 = multi.solve(bv, tol=1e-10, max_iter=5000, var=True)
            assert i1["converged"] == 1
            same_info(i1, i2)
            assert torch.equal(x1, x2) and torch.equal(v1, v2), (name, reuse)
        g1, gv1, j1 = one.backward(x1, b, tol=1e-12)
        g2, gv2, j2 = multi.backward(x2, b, tol=1e-12)
        assert torch.equal(g1, g2) and torch.equal(gv1, gv2) and j1["sweeps"] == j2["sweeps"], (name, reuse)
        for tol, M in ((1e-10, 0), (1e-10, 1), (1e-300, 6), (1e-300, 7), (0.5, 5)):
            x1, i1 = one.solve(b, tol=tol, max_iter=M, check=False)
            x2, i2 = multi.solve(b, tol=tol, max_iter=M, check=False)
            same_info(i1, i2)
            assert torch.equal(x1, x2), (name, reuse, tol, M)


@pytest.mark.parametrize("name", ["grid_97x61", "er_3001"])
def test_errors_are_reported_alike(name):
    p = CASES[name]()
    one, multi = pair(p)
    bad = p.b.copy()
    bad[p.n // 2] = np.nan
    s1 = one.solve(dev(bad), tol=1e-10, max_iter=50, check=False)[1]["status"]
    s2 = multi.solve(dev(bad), tol=1e-10, max_iter=50, check=False)[1]["status"]
    assert s1 == s2 < 0
    # the handle still solves afterwards, and b = 0 converges at round 0
    x1, i1 = one.solve(dev(p.b), tol=1e-10, max_iter=500)
    x2, i2 = multi.solve(dev(p.b), tol=1e-10, max_iter=500)
    assert torch.equal(x1, x2) and i1["sweeps"] == i2["sweeps"]
    x, info = one.solve(torch.zeros(p.n, dtype=torch.float64, device=DEV), tol=1e-10, max_iter=5)
    assert info["converged"] == 1 and info["sweeps"] == 0 and float(x.abs().max()) == 0.0


def test_shared_chip_and_threads():
    """Solves on streams of their own, from several threads at once and beside other work that
    fills the chip: each one either gets its workgroups in time or takes the launch-per-sweep
    path, with the same bits."""
    p = CASES["grid3d_64"]()
    q = CASES["er_60000"]()
    want = {}
    for key, r in (("grid", p), ("er", q)):
        s = g.Solver(r.row_ptr, r.col, r.val, device=DEV, reuse_precision=False)
        want[key] = s.solve(dev(r.b), tol=1e-10, max_iter=2000)[0]
    a = torch.randn(8192, 8192, device=DEV)
    got, errors = {}, []

    def work(i, key, r):
        try:
            st = torch.cuda.Stream()
            with torch.cuda.stream(st):
                s = g.Solver(r.row_ptr, r.col, r.val, device=DEV, reuse_precision=False)
                b = dev(r.b)
                got[i] = [(key, s.solve(b, tol=1e-10, max_iter=2000)[0]) for _ in range(6)]
                st.synchronize()
        except Exception as e:  # reported by the main thread
            errors.append(e)

    jobs = [("grid", p), ("er", q), ("grid", p), ("er", q)]
    threads = [threading.Thread(target=work, args=(i, key, r)) for i, (key, r) in enumerate(jobs)]
    for t in threads:
        t.start()
    for _ in range(20):
        a = (a @ a) * 1e-3
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for res in got.values():
        for key, x in res:
            assert torch.equal(x, want[key]), key


def dense_checks(p, **kw):
    """The launch-per-sweep path with the inner solves checked every round, as the resident loop checks them."""
    return g.Solver(p.row_ptr, p.col, p.val, device=DEV, layout="compact", predict_all=True, **kw)


OUTER = {
    "grid_33x32": CASES["grid_33x32"],        # rows of 4 slots
    "grid3d_24": lambda: workloads.grid3d_problem(24, 79),  # rows of 6
    "er_3001": CASES["er_3001"],              # chains of 8
    "er_130003": lambda: workloads.er_problem(130003, 8, 94),  # 1024 lanes
    "grid_9x7": lambda: workloads.grid2d_problem(9, 7, 8),  # one workgroup
}


@pytest.mark.parametrize("name", sorted(OUTER))
@pytest.mark.parametrize("reuse", [False, True])
def test_fp32_refinement_bitwise(name, reuse):
    p = OUTER[name]()
    rng = np.random.default_rng(6)
    for kw in ({}, {"check_every": 3}, {"inner_max_iter": 3, "max_outer": 5000}):
        one = g.Solver(p.row_ptr, p.col, p.val, device=DEV, precision="fp32", reuse_precision=reuse, **kw)
        multi = dense_checks(p, precision="fp32", reuse_precision=reuse, **kw)
        for bv in (dev(p.b), dev(rng.standard_normal(p.n))):  # with reuse, the second starts frozen
            x1, i1 = one.solve(bv, tol=1e-10, max_iter=100000)
            x2, i2 = multi.solve(bv, tol=1e-10, max_iter=100000)
            assert i1["converged"] == 1 and i1["outer_iters"] == i2["outer_iters"]
            same_info(i1, i2)
            assert torch.equal(x1, x2), (name, kw)
        x1, i1 = one.solve(dev(p.b), tol=1e-300, max_iter=7, check=False)
        x2, i2 = multi.solve(dev(p.b), tol=1e-300, max_iter=7, check=False)
        same_info(i1, i2)
        assert torch.equal(x1, x2)


@pytest.mark.parametrize("n", [500, 3000])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_loading_loops_bitwise(n, precision):
    p = workloads.config5(n=n, rows=2 * n)
    b = dev(p.b)
    for kw in ({"inner_tol": 1e-2, "reuse_precision": False}, {"inner_tol": 1e-2},
               {"inner_tol": 1e-3, "single_loop": True, "damping": 0.5},
               {"inner_tol": 1e-3, "single_loop": True, "damping": 1.0}):
        kw = dict(kw, precision=precision, gamma=-1.0, max_outer=5000)
        one = g.Solver(p.row_ptr, p.col, p.val, device=DEV, **kw)
        multi = dense_checks(p, **kw)
        for _ in range(2):
            x1, i1 = one.solve(b, tol=1e-9, max_iter=200000)
            x2, i2 = multi.solve(b, tol=1e-9, max_iter=200000)
            assert i1["converged"] == 1 and i1["outer_iters"] == i2["outer_iters"]
            same_info(i1, i2)
            assert torch.equal(x1, x2), kw


def test_loading_errors_are_reported_alike():
    p = workloads.config5(n=3000, rows=6000)  # diverges without loading
    one = g.Solver(p.row_ptr, p.col, p.val, device=DEV, precision="fp32")
    multi = dense_checks(p, precision="fp32")
    s1 = one.solve(dev(p.b), tol=1e-9, max_iter=5000, check=False)[1]
    s2 = multi.solve(dev(p.b), tol=1e-9, max_iter=5000, check=False)[1]
    assert s1["status"] == s2["status"] < 0
    x, info = one.solve(torch.zeros(p.n, dtype=torch.float64, device=DEV), tol=1e-9, max_iter=50)
    assert info["converged"] == 1 and float(x.abs().max()) == 0.0


SERIAL = ["grid_33x32", "grid_181x173", "grid3d_11", "grid3d_64", "er_3001", "er_60000", "er_isolated", "star_96", "tree"]


@pytest.mark.parametrize("name", SERIAL)
@pytest.mark.parametrize("check_every", [1, 3])
def test_serial_sweeps_bitwise(name, check_every):
    p = CASES[name]()
    one, multi = (g.Solver(p.row_ptr, p.col, p.val, device=DEV, layout="serial", check_every=check_every, **kw)
                  for kw in ({}, {"multi_launch": True}))
    b = dev(p.b)
    for tol, M in ((0, 0), (0, 1), (0, 2), (0, 7), (1e-10, 0), (1e-10, 1), (1e-300, 6), (1e-300, 7), (0.5, 5),
                   (1e-10, 3000)):
        x1, i1, v1 = one.solve(b, tol=tol, max_iter=M, var=True, check=False)
        x2, i2, v2 = multi.solve(b, tol=tol, max_iter=M, var=True, check=False)
        same_info(i1, i2)
        assert torch.equal(x1, x2) and torch.equal(v1, v2), (name, tol, M)
    assert i1["converged"] == 1
    g1, gv1, j1 = one.backward(x1, b, tol=1e-12)
    g2, gv2, j2 = multi.backward(x2, b, tol=1e-12)
    assert torch.equal(g1, g2) and torch.equal(gv1, gv2) and j1["sweeps"] == j2["sweeps"]


@pytest.mark.parametrize("name", ["grid_33x32", "grid3d_24", "er_3001", "btb"])
def test_serial_refinement_and_loading_bitwise(name):
    if name == "btb":
        p, kw = workloads.config5(n=1500, rows=3000), {"gamma": -1.0, "inner_tol": 1e-2, "max_outer": 5000}
    else:
        p, kw = OUTER.get(name, CASES.get(name))(), {}
    for prec in ("fp32", "fp64") if name == "btb" else ("fp32",):
        for extra in ({}, {"inner_max_iter": 3}):
            one, multi = (g.Solver(p.row_ptr, p.col, p.val, device=DEV, layout="serial", precision=prec,
                                   **dict(kw, max_outer=5000), **extra, **m) for m in ({}, {"multi_launch": True}))
            x1, i1 = one.solve(dev(p.b), tol=1e-9, max_iter=200000)
            x2, i2 = multi.solve(dev(p.b), tol=1e-9, max_iter=200000)
            same_info(i1, i2)
            assert i1["outer_iters"] == i2["outer_iters"] and torch.equal(x1, x2), (prec, extra)
