"""Timed cases of the GaBP library: what programs have it do, through its public entry points.

Five families cover the entry points.  "solve" is one right-hand side on a
handle that the program keeps (several graphs, precisions, layouts, with and
without the reuse of frozen precisions and the variances).  "adjoint" is a
training step through the autograd function, forward and backward.  "noalloc"
is the call of a serving loop that keeps no handle.  "loaded" solves systems
on which plain GaBP diverges, by the loading loops or through the augmented
matrix.  "batch" is many uneven systems with several right-hand sides each.

Every input is drawn from the seed on the GPU: off-diagonal values per
undirected edge and mirrored, diagonal = ratio * sum |A_ij|, right-hand sides
N(0, 1).
"""
import math

import torch

import paper_0811_2518_amd as gabp

DEV = "cuda"
TOL = 1e-10


def listed():
    return [
        # one small system whose matrix is new on every call, served without a handle
        {"name": "noalloc_er_600", "family": "noalloc", "graph": "er", "n": 600, "degree": 6, "ratio": 1.2},
        # the 32 x 32 grid of the benchmark, one right-hand side at a time
        {"name": "grid32_fp64", "family": "solve", "graph": "grid2d", "px": 32, "py": 32, "ratio": 1.2,
         "precision": "fp64", "layout": "auto", "reuse": False, "var": False},
        # a small grid solved for one right-hand side after another on a default handle
        {"name": "grid29x23_reuse", "family": "solve", "graph": "grid2d", "px": 29, "py": 23, "ratio": 1.1,
         "precision": "fp64", "layout": "auto", "reuse": True, "var": False},
        # a ragged mid-sized grid with marginal variances
        {"name": "grid181x173_var", "family": "solve", "graph": "grid2d", "px": 181, "py": 173, "ratio": 1.2,
         "precision": "fp64", "layout": "auto", "reuse": False, "var": True},
        # a sparse random graph of moderate size, many right-hand sides over time
        {"name": "er_30011_reuse", "family": "solve", "graph": "er", "n": 30011, "degree": 8, "ratio": 1.1,
         "precision": "fp64", "layout": "auto", "reuse": True, "var": False},
        # FP32 messages with FP64 refinement, the faster precision of the larger solves
        {"name": "er_130003_fp32", "family": "solve", "graph": "er", "n": 130003, "degree": 8, "ratio": 1.1,
         "precision": "fp32", "layout": "auto", "reuse": False, "var": False},
        # the colour-serial schedule, the fastest one on grids
        {"name": "grid3d_47_serial", "family": "solve", "graph": "grid3d", "px": 47, "ratio": 1.1,
         "precision": "fp64", "layout": "serial", "reuse": True, "var": False},
        # a training step on the benchmark's 64^3 grid: solve, loss, gradients on b and on A
        {"name": "adjoint_grid3d_64", "family": "adjoint", "graph": "grid3d", "px": 64, "ratio": 1.1},
        # hubs: the heavy-tailed degrees of web and social graphs
        {"name": "powerlaw_250007", "family": "solve", "graph": "powerlaw", "n": 250007, "degree": 8, "ratio": 1.1,
         "precision": "fp64", "layout": "auto", "reuse": False, "var": False},
        # the headline graph of the benchmark
        {"name": "er_1048576_fp64", "family": "solve", "graph": "er", "n": 1 << 20, "degree": 8, "ratio": 1.1,
         "precision": "fp64", "layout": "auto", "reuse": False, "var": False},
        # least squares: B^T B + 0.1 I, on which plain GaBP diverges, automatic loading
        {"name": "btb_30000_loaded", "family": "loaded", "method": "double", "n": 30000, "precision": "fp32"},
        # an uneven batch: grids and random graphs, 1 to 16 right-hand sides each
        {"name": "batch_192", "family": "batch", "systems": 192, "nmax": 16384, "kmax": 16, "layout": "auto"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["noalloc", "solve", "solve", "solve", "solve", "solve", "adjoint", "loaded", "batch"])
    ratio = rng.choice([1.1, 1.15, 1.2, 1.3])
    if kind == "noalloc":
        n, degree = _log_int(rng, 40, 1000), rng.randint(3, 8)
        return {"family": "noalloc", "graph": "er", "n": n, "degree": min(degree, 4000 // n), "ratio": ratio}
    if kind == "adjoint":
        return {"family": "adjoint", "graph": "grid3d", "px": _log_int(rng, 8, 64), "ratio": ratio}
    if kind == "loaded":
        method = rng.choice(["double", "single", "augmented"])
        return {"family": "loaded", "method": method, "n": _log_int(rng, 2000, 12000 if method == "augmented" else 30000),
                "precision": rng.choice(["fp64", "fp32"])}
    if kind == "batch":
        return {"family": "batch", "systems": _log_int(rng, 16, 192), "nmax": _log_int(rng, 500, 16384),
                "kmax": rng.randint(1, 16), "layout": rng.choice(["auto", "serial"])}
    graph = rng.choice(["grid2d", "grid3d", "er", "powerlaw"])
    c = {"family": "solve", "graph": graph}
    if graph == "grid2d":
        c["px"], c["py"] = _log_int(rng, 12, 500), _log_int(rng, 12, 500)
    elif graph == "grid3d":
        c["px"] = _log_int(rng, 6, 64)
    else:
        c["n"], c["degree"] = _log_int(rng, 300, 1 << 19 if graph == "er" else 250007), rng.randint(4, 12)
    c["ratio"] = ratio
    c["precision"] = rng.choice(["fp64", "fp64", "fp32"])
    c["layout"] = "auto" if graph == "powerlaw" else rng.choice(["auto", "auto", "serial"])
    c["reuse"] = rng.choice([False, True])
    c["var"] = c["precision"] == "fp64" and rng.random() < 0.3
    return c


# ---- inputs -----------------------------------------------------------------

def _grid_edges(dims):
    idx = torch.arange(math.prod(dims), device=DEV).reshape(dims)
    u, v = [], []
    for ax in range(len(dims)):
        u.append(idx.narrow(ax, 0, dims[ax] - 1).reshape(-1))
        v.append(idx.narrow(ax, 1, dims[ax] - 1).reshape(-1))
    return torch.cat(u), torch.cat(v)


def _distinct(n, m, pick):
    """m distinct undirected pairs from pick(count) -> (u, v), u != v."""
    m = min(m, n * (n - 1) // 4)
    keys = torch.empty(0, dtype=torch.int64, device=DEV)
    while keys.numel() < m:
        u, v = pick(int((m - keys.numel()) * 1.2) + 64)
        k = torch.minimum(u, v) * n + torch.maximum(u, v)
        keys = torch.unique(torch.cat([keys, k[u != v]]))
    # thin evenly to m, so that no part of the graph is favoured
    keys = keys[(torch.arange(m, device=DEV) * keys.numel()) // m]
    return keys // n, keys % n


def _edges(c, gen):
    """(n, u, v, w) of a case's graph."""
    graph = c["graph"]
    if graph in ("grid2d", "grid3d"):
        dims = [c["py"], c["px"]] if graph == "grid2d" else [c["px"]] * 3
        n = math.prod(dims)
        u, v = _grid_edges(dims)
        w = -torch.rand(u.numel(), generator=gen, device=DEV, dtype=torch.float64)
        return n, u, v, w if graph == "grid2d" else w * 0.9 - 0.1
    n = c["n"]
    if graph == "er":
        def pick(k):
            return torch.randint(0, n, (2, k), generator=gen, device=DEV).unbind(0)
    else:  # Chung-Lu pairs, degree exponent 2.1, labels shuffled
        cdf = torch.cumsum((torch.arange(n, device=DEV, dtype=torch.float64) + 1.0) ** (-1.0 / 1.1), 0)
        label = torch.randperm(n, generator=gen, device=DEV)

        def pick(k):
            q = torch.rand(2, k, generator=gen, device=DEV, dtype=torch.float64) * cdf[-1]
            return label[torch.searchsorted(cdf, q).clamp_(max=n - 1)].unbind(0)
    u, v = _distinct(n, c["degree"] * n // 2, pick)
    return n, u, v, torch.randn(u.numel(), generator=gen, device=DEV, dtype=torch.float64)


def _csr(n, u, v, w, ratio):
    """Full symmetric CSR (int32, int32, float64) from undirected pairs."""
    rows = torch.cat([u, v, torch.arange(n, device=DEV)])
    cols = torch.cat([v, u, torch.arange(n, device=DEV)])
    order = torch.argsort(rows * n + cols)
    rows, cols = rows[order], cols[order]
    val = torch.cat([w, w, torch.zeros(n, device=DEV, dtype=torch.float64)])[order]
    cnt = torch.bincount(rows, minlength=n)
    absum = torch.segment_reduce(val.abs(), "sum", lengths=cnt)
    diag = torch.where(absum > 0, ratio * absum, torch.ones_like(absum))
    val = torch.where(rows == cols, diag[rows], val)
    ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(cnt, 0, out=ptr[1:])
    return ptr.to(torch.int32), cols.to(torch.int32), val


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _system(c, gen):
    n, u, v, w = _edges(c, gen)
    ptr, col, val = _csr(n, u, v, w, c["ratio"])
    return n, ptr, col, val


def _rect(c, gen):
    """B (2n x n), 4 distinct N(0, 1) entries per row, as sorted columns and values [2n, 4]."""
    n, m = c["n"], 2 * c["n"]
    # distinct by construction: one column from each quarter of the range
    quarter = torch.arange(4, device=DEV) * (n // 4)
    cols = quarter + torch.randint(0, n // 4, (m, 4), generator=gen, device=DEV)
    # every row shifted cyclically, so that no column is tied to one quarter
    cols, order = torch.sort((cols + torch.randint(0, n, (m, 1), generator=gen, device=DEV)) % n, dim=1)
    vals = torch.randn(m, 4, generator=gen, device=DEV, dtype=torch.float64)
    return n, m, cols, torch.gather(vals, 1, order)


def _normal_matrix(n, cols, vals):
    """A = B^T B + 0.1 I in CSR; every sum is formed in one fixed order."""
    keys = (cols[:, :, None] * n + cols[:, None, :]).reshape(-1)
    prod = (vals[:, :, None] * vals[:, None, :]).reshape(-1)
    eye = torch.arange(n, device=DEV) * (n + 1)
    keys = torch.cat([keys, eye])
    prod = torch.cat([prod, torch.full((n,), 0.1, device=DEV, dtype=torch.float64)])
    keys, order = torch.sort(keys, stable=True)
    uniq, cnt = torch.unique_consecutive(keys, return_counts=True)
    val = torch.segment_reduce(prod[order], "sum", lengths=cnt)
    ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(uniq // n, minlength=n), 0, out=ptr[1:])
    return ptr.to(torch.int32), (uniq % n).to(torch.int32), val


def _batch(c, gen):
    """Block-diagonal CSR of uneven systems and their right-hand sides.

    The sizes belong to the case; the graphs' edges, the values and B to the seed."""
    host = torch.Generator().manual_seed(2521)
    S = c["systems"]
    kinds = torch.randint(0, 3, (S,), generator=host).tolist()
    sizes = torch.exp(torch.rand(S, generator=host) * math.log(c["nmax"] / 64.0)).mul(64.0).tolist()
    ratios = (1.05 + 0.45 * torch.rand(S, generator=host)).tolist()
    nrhs = torch.randint(1, c["kmax"] + 1, (S,), generator=host).tolist()
    degrees = torch.randint(4, 13, (S,), generator=host).tolist()
    us, vs, ws, rat, off = [], [], [], [], [0]
    for s in range(S):
        if kinds[s] == 0:
            side = max(2, round(math.sqrt(sizes[s])))
            sub = {"graph": "grid2d", "px": side, "py": side}
        elif kinds[s] == 1:
            sub = {"graph": "grid3d", "px": max(2, round(sizes[s] ** (1.0 / 3.0)))}
        else:
            sub = {"graph": "er", "n": round(sizes[s]), "degree": degrees[s]}
        n, u, v, w = _edges(sub, gen)
        us.append(u + off[-1])
        vs.append(v + off[-1])
        ws.append(w)
        rat.append(torch.full((n,), ratios[s], device=DEV, dtype=torch.float64))
        off.append(off[-1] + n)
    ptr, col, val = _csr(off[-1], torch.cat(us), torch.cat(vs), torch.cat(ws), torch.cat(rat))
    rhs_off = [0]
    for s in range(S):
        rhs_off.append(rhs_off[-1] + (off[s + 1] - off[s]) * nrhs[s])
    B = torch.randn(rhs_off[-1], generator=gen, device=DEV, dtype=torch.float64)
    return off, ptr, col, val, nrhs, rhs_off, B


# ---- what a program holds, and one pass -------------------------------------

def prepare(case, seed):
    gen = _gen(seed)
    fam = case["family"]
    st = {"family": fam, "case": case}
    if fam == "batch":
        off, ptr, col, val, nrhs, rhs_off, B = _batch(case, gen)
        st["solver"] = gabp.BatchedSolver(off, ptr, col, val, layout=case["layout"])
        st.update(nrhs=nrhs, rhs_off=rhs_off, B=B)
        return st
    if fam == "loaded":
        n, m, cols, vals = _rect(case, gen)
        if case["method"] == "augmented":
            ptr = torch.arange(m + 1, device=DEV, dtype=torch.int32) * 4
            d = torch.full((n,), 0.1, device=DEV, dtype=torch.float64)
            st["solver"] = gabp.AugmentedSolver(m, n, ptr, cols.reshape(-1).to(torch.int32), vals.reshape(-1), d, 1.0,
                                                precision=case["precision"], inner_tol=1e-2, inner_max_iter=2000,
                                                max_outer=5000)
        else:
            ptr, col, val = _normal_matrix(n, cols, vals)
            single = case["method"] == "single"
            st["solver"] = gabp.Solver(ptr, col, val, precision=case["precision"], gamma=-1.0, single_loop=single,
                                       damping=1.0, inner_tol=1e-3 if single else 1e-2,
                                       inner_max_iter=20000 if single else 2000, max_outer=5000,
                                       reuse_precision=False)
        st["b"] = torch.randn(n, generator=gen, device=DEV, dtype=torch.float64)
        return st
    n, ptr, col, val = _system(case, gen)
    st["b"] = torch.randn(n, generator=gen, device=DEV, dtype=torch.float64)
    if fam == "noalloc":
        st.update(ptr=ptr, col=col, val=val)
    elif fam == "adjoint":
        st["target"] = torch.randn(n, generator=gen, device=DEV, dtype=torch.float64)
        st["solver"] = gabp.Solver(ptr, col, val)
        st["vals"] = val.requires_grad_(True)
        st["b"].requires_grad_(True)
    else:
        st["solver"] = gabp.Solver(ptr, col, val, precision=case["precision"], layout=case["layout"],
                                   reuse_precision=case["reuse"])
    return st


def run(st):
    fam, case = st["family"], st["case"]
    if fam == "noalloc":
        x, info = gabp.binding.solve_noalloc(st["ptr"], st["col"], st["val"], st["b"], tol=TOL)
        return {"x": x, "converged": info["converged"]}
    if fam == "solve":
        out = st["solver"].solve(st["b"], tol=TOL, var=case["var"])
        got = {"x": out[0], "converged": out[1]["converged"]}
        if case["var"]:
            got["var"] = out[2]
        return got
    if fam == "adjoint":
        x = gabp.gabp_solve(st["solver"], st["vals"], st["b"], TOL, 5000)
        loss = 0.5 * (x - st["target"]).square().sum()
        grad_vals, grad_b = torch.autograd.grad(loss, (st["vals"], st["b"]))
        return {"x": x.detach(), "grad_vals": grad_vals, "grad_b": grad_b}
    if fam == "loaded":
        if case["method"] == "augmented":
            x, info = st["solver"].solve_blocks(b=st["b"], tol=TOL)
        else:
            x, info = st["solver"].solve(st["b"], tol=TOL, max_iter=100000)
        return {"x": x, "converged": info["converged"]}
    X, infos, status = st["solver"].solve(st["nrhs"], st["rhs_off"], st["B"], tol=TOL)
    return {"X": X, "status": status}


# ---- what a pass cannot do without ------------------------------------------

def _sweeps(graph, ratio):
    """About the sweeps to 1e-10: attractive grids contract by 1 / ratio^2 a sweep, random signs faster."""
    return 11.5 / math.log(ratio) if graph in ("grid2d", "grid3d") else 23.0


def _size(c):
    """(rows, directed slots) of a case's graph."""
    if c["graph"] == "grid2d":
        px, py = c["px"], c["py"]
        return px * py, 2 * (px * (py - 1) + py * (px - 1))
    if c["graph"] == "grid3d":
        p = c["px"]
        return p ** 3, 6 * p * p * (p - 1)
    return c["n"], c["degree"] * c["n"]


def work(case):
    # the matrix (column and value per slot; row pointer and diagonal per row),
    # right-hand sides and solutions once; about 14 operations per slot and sweep
    fam = case["family"]
    if fam == "batch":
        n = (case["nmax"] - 64.0) / math.log(case["nmax"] / 64.0) * case["systems"]
        E, k = 6.5 * n, (case["kmax"] + 1) / 2.0
        return {"bytes": 12 * E + 12 * n + 16 * n * k, "flops": 5 * 60 * E * k}
    if fam == "loaded":
        n = case["n"]
        E = 16 * n if case["method"] == "augmented" else 24 * n
        return {"bytes": 12 * E + 28 * n, "flops": 14 * 1000 * E}
    n, E = _size(case)
    sweeps = _sweeps(case["graph"], case["ratio"])
    solve = {"bytes": 12 * E + 28 * n, "flops": 14 * sweeps * E}
    if fam == "adjoint":
        return {"bytes": 2 * solve["bytes"] + 8 * (E + n) + 16 * n, "flops": 2 * solve["flops"] + 4 * E}
    if case.get("var"):
        solve["bytes"] += 8 * n
    return solve


# ---- the same values in 64 bits, by conjugate gradients ---------------------

def _cg(apply, diag, b, iters=1500):
    """Jacobi-preconditioned CG to the rounding floor, restarted once from its own residual."""
    x = torch.zeros_like(b)
    for _ in range(2):
        r = b - apply(x)
        if float(r.norm()) == 0.0:
            break
        z = r / diag
        p, rz = z.clone(), torch.dot(r, z)
        stop = 1e-14 * float(r.norm())
        for it in range(iters):
            q = apply(p)
            a = rz / torch.dot(p, q)
            x = x + a * p
            r = r - a * q
            if it % 10 == 9 and not float(r.norm()) > stop:
                break
            z = r / diag
            rz, old = torch.dot(r, z), rz
            p = z + (rz / old) * p
    return x


def _rows(ptr):
    return torch.repeat_interleave(torch.arange(ptr.numel() - 1, device=DEV), (ptr[1:] - ptr[:-1]).long())


def _operator(ptr, col, val):
    n = ptr.numel() - 1
    A = torch.sparse_csr_tensor(ptr, col, val, size=(n, n))
    diag = val[_rows(ptr) == col]
    return (lambda x: A @ x), diag


def exact(case, seed):
    gen = _gen(seed)
    fam = case["family"]
    if fam == "batch":
        off, ptr, col, val, nrhs, rhs_off, B = _batch(case, gen)
        rows, cols = _rows(ptr), col.long()
        # one unknown for every row and right-hand side, numbered as B is
        o = torch.tensor(off, device=DEV)
        k = torch.tensor(nrhs, device=DEV)
        base = torch.tensor(rhs_off, device=DEV)
        sys_of = torch.searchsorted(o, rows, right=True) - 1
        rep = k[sys_of]
        j = torch.arange(int(rep.sum()), device=DEV) - torch.repeat_interleave(torch.cumsum(rep, 0) - rep, rep)
        big_r = torch.repeat_interleave(base[sys_of] + (rows - o[sys_of]) * rep, rep) + j
        big_c = torch.repeat_interleave(base[sys_of] + (cols - o[sys_of]) * rep, rep) + j
        big_v = torch.repeat_interleave(val, rep)
        order = torch.argsort(big_r, stable=True)
        big_ptr = torch.zeros(rhs_off[-1] + 1, dtype=torch.int64, device=DEV)
        torch.cumsum(torch.bincount(big_r, minlength=rhs_off[-1]), 0, out=big_ptr[1:])
        apply, diag = _operator(big_ptr.to(torch.int32), big_c[order].to(torch.int32), big_v[order])
        return {"X": _cg(apply, diag, B), "status": None}
    if fam == "loaded":
        n, m, cols, vals = _rect(case, gen)
        b = torch.randn(n, generator=gen, device=DEV, dtype=torch.float64)
        apply, diag = _operator(*_normal_matrix(n, cols, vals))
        return {"x": _cg(apply, diag, b), "converged": None}
    n, ptr, col, val = _system(case, gen)
    b = torch.randn(n, generator=gen, device=DEV, dtype=torch.float64)
    apply, diag = _operator(ptr, col, val)
    x = _cg(apply, diag, b)
    if fam == "adjoint":
        target = torch.randn(n, generator=gen, device=DEV, dtype=torch.float64)
        lam = _cg(apply, diag, x - target)
        rows, cols = _rows(ptr), col.long()
        grad = -torch.where(rows == cols, lam[rows] * x[rows], lam[rows] * x[cols] + lam[cols] * x[rows])
        return {"x": x, "grad_vals": grad, "grad_b": lam}
    got = {"x": x, "converged": None}
    if case.get("var"):
        got["var"] = None  # the marginal precisions of GaBP are its own, not those of A
    return got
