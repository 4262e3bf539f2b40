"""Performance cases: the calls a program makes to this library, over the sizes it makes them at.

A case is one public call (or the call pair of a training step) on one matrix family:

    call     symbolic       Phase I: pattern of F, then the arrays a caller exports from it
             numeric        Phase II with its default zero-pivot report
             apply          y = M^-1 b, what every outer solver calls per iteration
             gmres          a whole preconditioned solve by substitution
             gmres_inverse  the same with the incomplete inverses (two products)
             inverse        building the incomplete inverses from a factor
             batched        one launch of the captured factor + solve of a batch
             reverse        ILUApply forward and backward: y, d/d(values of A), d/db
    matrix   2d5 / 3d7      5- and 7-point convection-diffusion on m x m / m x m x m
             3d27           27-point stencil on m x m x m
             banded         random banded, 8 columns within 2,000 of the diagonal and 2 anywhere
    size     m, or the number of rows of a banded matrix
    k        level of fill
    batch    instances sharing the pattern (1: a single matrix, one-dimensional values)

``exact`` is plain Python and numpy in 64 bits: rows merged in order for the
pattern, the textbook elimination, substitutions, reverse sweep and GMRES.
"""
import math

import numpy as np
import torch

from paper_0803_0048_amd import binding as T
from paper_0803_0048_amd import inputs

# entries of A, entries of F and updates of the elimination per row, away from the boundary
PER_ROW = {
    "2d5": [(5, 5, 2), (5, 7, 7), (5, 9, 12), (5, 13, 27)],
    "3d7": [(7, 7, 3), (7, 13, 20), (7, 22, 63), (7, 41, 214)],
    "3d27": [(26, 26, 85), (26, 59, 446), (26, 106, 1350)],
    "banded": [(11, 11, 0.1), (11, 37, 15), (11, 165, 280)],
}


def _case(name, call, matrix, size, k, batch=1):
    return {"name": name, "call": call, "matrix": matrix, "size": size, "k": k, "batch": batch}


def listed():
    return [
        # the smallest problem in earnest (4,096 rows): one preconditioner application inside
        # another package's solver, the refactorisation after a change of coefficients, a whole solve
        _case("apply_2d_64_ilu1", "apply", "2d5", 64, 1),
        _case("numeric_2d_64_ilu1", "numeric", "2d5", 64, 1),
        _case("gmres_2d_64_ilu1", "gmres", "2d5", 64, 1),
        # 3-D stencils: wide dependency levels, short rows (7-point) and longer ones (27-point)
        _case("apply_3d_64_ilu1", "apply", "3d7", 64, 1),
        _case("numeric_3d27_50_ilu1", "numeric", "3d27", 50, 1),
        # the headline general sparse matrix, every phase: deep, narrow dependency graphs
        _case("symbolic_banded_160000_ilu2", "symbolic", "banded", 160000, 2),
        _case("numeric_banded_160000_ilu2", "numeric", "banded", 160000, 2),
        _case("apply_banded_160000_ilu2", "apply", "banded", 160000, 2),
        _case("inverse_banded_160000_ilu2", "inverse", "banded", 160000, 2),
        _case("gmres_inverse_banded_160000_ilu2", "gmres_inverse", "banded", 160000, 2),
        # time stepping of many small systems of one pattern, replayed from a graph
        _case("batched_2d_128_x256_ilu2", "batched", "2d5", 128, 2, 256),
        # a training step through the preconditioner
        _case("reverse_3d_32_x16_ilu1", "reverse", "3d7", 32, 1, 16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["symbolic", "numeric", "apply", "apply", "gmres", "gmres_inverse", "inverse", "batched",
                       "reverse"])
    batch = 1
    if call == "batched":
        matrix = rng.choice(["2d5", "3d7"])
        size = _log_int(rng, 12, 128) if matrix == "2d5" else _log_int(rng, 6, 24)
        k = rng.randint(0, 2)
        batch = _log_int(rng, 3, 256)
    elif call == "reverse":
        matrix = rng.choice(["2d5", "3d7"])
        size = _log_int(rng, 12, 150) if matrix == "2d5" else _log_int(rng, 6, 32)
        k = rng.randint(0, 1)
        batch = rng.randint(1, 16)
    elif call == "gmres_inverse":
        matrix, size, k = "banded", _log_int(rng, 3000, 160000), rng.randint(1, 2)
    else:
        matrix = rng.choice(["2d5", "3d7", "3d27", "banded"])
        if matrix == "2d5":
            size, k = _log_int(rng, 16, 100 if call == "gmres" else 400), rng.randint(0, 3)
        elif matrix == "3d7":
            size, k = _log_int(rng, 8, 64), rng.randint(0, 2)
        elif matrix == "3d27":
            size, k = _log_int(rng, 6, 50), rng.randint(0, 1)
        else:
            size, k = _log_int(rng, 2000, 160000), rng.randint(0, 2)
    c = _case("", call, matrix, size, k, batch)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _cut(A, rng):
    """A with one in a hundred of its off-diagonal entries (drawn anywhere) left out."""
    rows = np.repeat(np.arange(A.n), np.diff(A.rowptr))
    off = np.flatnonzero(rows != A.col)
    keep = np.ones(A.nnz, dtype=bool)
    keep[rng.choice(off, size=max(1, off.size // 100), replace=False)] = False
    rowptr = np.zeros(A.n + 1, dtype=np.int64)
    np.cumsum(np.bincount(rows[keep], minlength=A.n), out=rowptr[1:])
    return inputs.CSR(A.n, rowptr, A.col[keep], A.val[keep])


def _matrix(case, seed):
    """CSR matrix and right-hand side (host), values [nnz] or [nnz, batch].  A size has one
    structure, its values drawn anew; the symbolic phase, which reads no values, gets its
    structure from the seed."""
    rng = np.random.default_rng(seed)
    m, B = case["size"], case["batch"]
    if case["matrix"] == "banded":
        A = inputs.random_banded(m, seed if case["call"] == "symbolic" else 1002)
        diag = A.col == np.repeat(np.arange(m), np.diff(A.rowptr))
        A.val = rng.uniform(-1.0, 1.0, size=A.nnz)
        A.val[diag] = 0.0
        A.val[diag] = 1.1 * np.abs(A.val).reshape(m, -1).sum(axis=1)
    elif case["matrix"] == "3d27":
        A = inputs.stencil27_3d(m, 1.0, rng.uniform(-10.0, 10.0, size=3))
    elif case["matrix"] == "2d5":
        if B > 1:
            bx, by = rng.uniform(-50.0, 50.0, size=(2, B))
            A = inputs.conv_diff_2d(m, rng.uniform(0.5, 2.0, size=B), bx, by)
        else:
            A = inputs.conv_diff_2d(m, 1.0, *rng.uniform(-20.0, 20.0, size=2))
    elif B > 1:
        A = inputs.conv_diff_3d(m, rng.uniform(0.5, 2.0, size=B), rng.uniform(-50.0, 50.0, size=(B, 3)))
    else:  # cell Peclet numbers up to 1.5, as the single 64^3 problem of inputs.py has, at every m
        A = inputs.conv_diff_3d(m, 1.0, rng.uniform(-3.0, 3.0, size=3) * (m + 1))
    if case["call"] == "symbolic" and case["matrix"] != "banded":
        A = _cut(A, rng)
    shape = (A.n,) if B == 1 else (A.n, B)
    return A, rng.standard_normal(shape), rng.standard_normal(shape)


def prepare(case, seed):
    A, b, t = _matrix(case, seed)
    dev = torch.device("cuda")
    s = {"call": case["call"], "k": case["k"], "rowptr": torch.from_numpy(A.rowptr).to(dev),
         "col": torch.from_numpy(A.col).to(dev)}
    if case["call"] == "symbolic":
        # the caller's own arrays for the columns and levels of F, with room to spare (their
        # length is known only after the call)
        room = A.n * (PER_ROW[case["matrix"]][case["k"]][1] * 5 // 4 + 1)
        s["colF"] = torch.full((room,), -1, dtype=torch.int32, device=dev)
        s["levF"] = torch.zeros(room, dtype=torch.uint8, device=dev)
        return s
    s["a"], s["b"] = torch.from_numpy(A.val).to(dev), torch.from_numpy(b).to(dev)
    s["pat"] = T.symbolic(s["rowptr"], s["col"], case["k"])
    if case["call"] == "batched":
        s["graph"] = T.BatchedGraph(s["pat"], s["a"], s["b"])
    elif case["call"] == "reverse":
        s["t"] = torch.from_numpy(t).to(dev)
    elif case["call"] != "numeric":
        s["f"] = T.numeric(s["pat"], s["a"])
        if case["call"] == "gmres_inverse":
            s["f"] = T.inverse(s["pat"], s["f"])
    return s


def run(s):
    call = s["call"]
    if call == "symbolic":
        s["pat"] = T.symbolic(s["rowptr"], s["col"], s["k"])
        p, info = s["pat"].export(), s["pat"].info
        s["colF"][:info["nnz_f"]] = p["col"]
        s["levF"][:info["nnz_f"]] = p["level"]
        return {"rowptr": p["rowptr"], "col": s["colF"], "diag": p["diag"], "level": s["levF"], "a2f": p["a2f"],
                **{f: info[f] for f in ("nnz_f", "nnz_l", "n_updates", "max_row", "depth_l", "depth_u")}}
    if call == "numeric":
        return T.numeric(s["pat"], s["a"])
    if call == "apply":
        return T.apply(s["pat"], s["f"], s["b"])
    if call == "inverse":
        return T.inverse(s["pat"], s["f"])
    if call == "batched":
        s["graph"].launch()
        return s["graph"].f_val, s["graph"].y
    if call == "reverse":
        a, b = s["a"].detach().requires_grad_(), s["b"].detach().requires_grad_()
        y = T.ILUApply.apply(a, b, s["pat"])
        loss = ((y - s["t"]) ** 2).sum()
        loss.backward()
        return y.detach(), a.grad, b.grad
    x, info = T.gmres(s["pat"], s["a"], s["f"], s["b"], inverse=call == "gmres_inverse")
    return {"x": x, "relres": info["relres"], "iters": info["iters"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    na, nf, nu = PER_ROW[case["matrix"]][case["k"]]
    n = case["size"] if case["matrix"] == "banded" else case["size"] ** (2 if case["matrix"] == "2d5" else 3)
    na, nf, nu, B = na * n, nf * n, nu * n, case["batch"]
    call = case["call"]
    factor = 4 * na + 4 * nf + 8 * (na + nf) * B  # maps, A read, F written
    solve = 4 * nf + 8 * nf * B + 3 * 8 * n * B  # F and its columns read; b, x, y
    if call == "symbolic":
        return {"bytes": 8 * na + 5 * nf + 20 * n, "flops": 0}
    if call == "numeric":
        return {"bytes": factor, "flops": (2 * nu + nf / 2) * B}
    if call == "apply":
        return {"bytes": solve, "flops": 2 * nf}
    if call == "inverse":
        return {"bytes": 4 * nf + 16 * nf, "flops": 2 * nu}
    if call == "batched":
        return {"bytes": factor + solve, "flops": (2 * nu + 2.5 * nf) * B}
    if call == "reverse":  # forward; both transposed solves; the reverse sweep reads F and F-bar, writes A-bar
        return {"bytes": factor + 2 * solve + 16 * nf * B + 8 * na * B, "flops": (6 * nu + 6 * nf) * B}
    iters = 8 if case["matrix"] == "banded" else max(4, case["size"] // (2 * case["k"] + 2)) \
        if case["matrix"] == "2d5" else 10
    return {"bytes": iters * (12 * nf + 12 * na + 16 * n * (iters % 30 // 2 + 4)),
            "flops": iters * (2 * nf + 2 * na + 4 * n * (iters % 30 // 2 + 2))}


# ---------------------------------------------------------------------------
# the same in plain Python; a value is a float or an array over the batch
# ---------------------------------------------------------------------------
def _pattern(A, k):
    """Per row a dict column -> level (rows merged in ascending order, levels <= k kept)."""
    rows = []
    for i in range(A.n):
        lev = dict.fromkeys(A.col[A.rowptr[i]:A.rowptr[i + 1]].tolist(), 0)
        todo, done = sorted(c for c in lev if c < i), set()
        while todo:
            h = todo.pop(0)
            done.add(h)
            for t, l in rows[h].items():
                if t > h and lev[h] + l + 1 <= k and lev[h] + l + 1 < lev.get(t, k + 1):
                    if t < i and t not in lev:
                        todo.append(t)
                        todo.sort()
                    lev[t] = lev[h] + l + 1
        rows.append(dict(sorted(lev.items())))
    return rows


def _factor(A, rows, vals):
    """Per row a dict column -> value of F = L + U - I."""
    F, upper = [], []
    for i, lev in enumerate(rows):
        w = dict.fromkeys(lev, vals[0] * 0.0)
        a, e = A.rowptr[i], A.rowptr[i + 1]
        w.update(zip(A.col[a:e].tolist(), vals[a:e]))
        for h in lev:
            if h >= i:
                break
            l = w[h] = w[h] / F[h][h]
            for t, u in upper[h]:
                if t in w:
                    w[t] = w[t] - l * u
        F.append(w)
        upper.append([(t, u) for t, u in w.items() if t > i])
    return F


def _solve(F, b):
    n = len(F)
    x, y = [None] * n, [None] * n
    for i in range(n):
        s = b[i]
        for h, f in F[i].items():
            if h >= i:
                break
            s = s - f * x[h]
        x[i] = s
    for i in range(n - 1, -1, -1):
        s = x[i]
        for j, f in reversed(F[i].items()):
            if j <= i:
                break
            s = s - f * y[j]
        y[i] = s / F[i][i]
    return x, y


def _inverse(F):
    """Incomplete inverses of L and U on F's pattern, per row a dict."""
    n = len(F)
    G = [dict.fromkeys(r, 0.0) for r in F]
    for i in range(n):
        for t, f in F[i].items():
            if t >= i:
                break
            G[i][t] = -f
        for h, f in F[i].items():
            if h >= i:
                break
            for t, g in G[h].items():
                if t >= h:
                    break
                if t in F[i]:
                    G[i][t] = G[i][t] - f * g
    for i in range(n - 1, -1, -1):
        acc = {t: 1.0 if t == i else 0.0 for t in F[i] if t >= i}
        for j, u in reversed(F[i].items()):
            if j <= i:
                break
            for t, g in G[j].items():
                if t >= j and t in acc:
                    acc[t] = acc[t] - u * g
        G[i].update({t: v / F[i][i] for t, v in acc.items()})
    return G


def _reverse(A, F, x, y, t):
    """Gradients of sum (y - t)^2 with respect to A's values and b."""
    n = len(F)
    zs, w = [2.0 * (y[i] - t[i]) for i in range(n)], None
    for i in range(n):  # U^T z = ybar, then L^T w = z
        zs[i] = zs[i] / F[i][i]
        for j, u in F[i].items():
            if j > i:
                zs[j] = zs[j] - u * zs[i]
    w = list(zs)
    for i in range(n - 1, -1, -1):
        for h, l in F[i].items():
            if h < i:
                w[h] = w[h] - l * w[i]
    g = [{c: -(w[i] * x[c]) if c < i else -(zs[i] * y[c]) for c in F[i]} for i in range(n)]
    for j in range(n - 1, -1, -1):
        for h in reversed([c for c in F[j] if c < j]):
            l, lb = F[j][h], g[j][h]
            for c, u in F[h].items():
                if c > h and c in g[j]:
                    lb = lb - g[j][c] * u
                    g[h][c] = g[h][c] - g[j][c] * l
            g[j][h] = lb / F[h][h]
            g[h][h] = g[h][h] - lb * l / F[h][h]
    abar = [g[i][c] for i in range(n) for c in A.col[A.rowptr[i]:A.rowptr[i + 1]].tolist()]
    return abar, w


def _gmres(A, precond, b, m=30, rtol=1e-8):
    rows = np.repeat(np.arange(A.n), np.diff(A.rowptr))
    mul = lambda v: np.bincount(rows, A.val * v[A.col], A.n)  # noqa: E731
    x, hist, tol = np.zeros(A.n), [], rtol * np.linalg.norm(b)
    while True:
        r = b - mul(x)
        beta = np.linalg.norm(r)
        if beta <= tol or len(hist) >= 10000:
            return {"x": x, "relres": beta / np.linalg.norm(b), "iters": len(hist)}
        V, H, g, rot = [r / beta], np.zeros((m + 1, m)), np.zeros(m + 1), []
        g[0] = beta
        for j in range(m):
            w = mul(precond(V[j]))
            for i in range(j + 1):
                H[i, j] = w @ V[i]
                w = w - H[i, j] * V[i]
            H[j + 1, j] = np.linalg.norm(w)
            V.append(w / H[j + 1, j])
            for i, (c, s) in enumerate(rot):
                H[i, j], H[i + 1, j] = c * H[i, j] + s * H[i + 1, j], c * H[i + 1, j] - s * H[i, j]
            rho = math.hypot(H[j, j], H[j + 1, j])
            rot.append((H[j, j] / rho, H[j + 1, j] / rho))
            H[j, j], H[j + 1, j] = rho, 0.0
            g[j], g[j + 1] = rot[j][0] * g[j], -rot[j][1] * g[j]
            hist.append(abs(g[j + 1]))
            if hist[-1] <= tol:
                break
        yv = np.linalg.solve(H[:j + 1, :j + 1], g[:j + 1])
        x = x + precond(sum(c * v for c, v in zip(yv, V)))


def exact(case, seed):
    na, nf, nu = PER_ROW[case["matrix"]][case["k"]]
    n = case["size"] if case["matrix"] == "banded" else case["size"] ** (2 if case["matrix"] == "2d5" else 3)
    steps = n * (nf * nf / 4 + nu)
    call = case["call"]
    if call == "gmres":
        steps += 40 * n * nf
    if call == "symbolic" or steps * (6 if case["batch"] > 1 else 1) > 1.8e7:
        return None  # whole numbers alone, or minutes of Python
    A, b, t = _matrix(case, seed)
    F = _factor(A, _pattern(A, case["k"]), list(A.val))
    flat = lambda rows: np.array([v for r in rows for v in r.values()])  # noqa: E731
    if call == "numeric":
        return flat(F)
    if call == "inverse":
        return flat(_inverse(F))
    if call == "gmres":
        return _gmres(A, lambda v: np.array(_solve(F, v)[1]), b)
    if call == "gmres_inverse":
        G = _inverse(F)
        rows, cols = np.repeat(np.arange(A.n), [len(r) for r in G]), np.array([c for r in G for c in r])
        lo, v = cols < rows, flat(G)
        return _gmres(A, lambda p: np.bincount(
            rows[~lo], v[~lo] * (p + np.bincount(rows[lo], v[lo] * p[cols[lo]], A.n))[cols[~lo]], A.n), b)
    x, y = _solve(F, list(b))
    if call == "apply":
        return np.array(y)
    if call == "batched":
        return flat(F), np.array(y)
    abar, bbar = _reverse(A, F, x, y, t)
    return np.array(y), np.array(abar), np.array(bbar)
