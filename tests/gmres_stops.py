"""GMRES that stops at a chosen step, against the oracle's bits: by the
tolerance, by maxit and by a breakdown, at every position of a cycle.  Run by
test_gpu_gmres_stops.py with the product library and by jitter_check_auto.py
with the race check build, where the host reads the report of a step only after
every step it has launched, the one launched ahead included, has reported."""
from __future__ import annotations

import numpy as np

import oracle as O
from paper_0803_0048_amd import binding as T
from paper_0803_0048_amd import inputs as I
from tests.gpu_util import assert_bits_equal, g

RESTART = 5
KINDS = ("tolerance", "maxit", "breakdown")


def _bidiagonal(n):
    """Ones on the diagonal and below: with M = I and b = e_0 the Krylov space
    grows by one coordinate a step, and step `block` of a chain that ends there
    finds nothing left (all values exact)."""
    rows = np.repeat(np.arange(n), 2)[1:]
    cols = np.stack([np.arange(n) - 1, np.arange(n)], 1).reshape(-1)[1:]
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(rows, minlength=n), out=rp[1:])
    return I.CSR(n, rp, cols.astype(np.int32), np.ones(rows.size))


def _same(got, info, ref, what):
    assert info["iters"] == ref["iters"], (what, info["iters"], ref["iters"])
    assert info["status"] == ref["status"], (what, info["status"], ref["status"])
    assert_bits_equal(np.array(info["hist"]), ref["hist"], f"{what}: history")
    assert_bits_equal(got, ref["x"], f"{what}: x")
    assert_bits_equal(np.array([info["relres"]]), np.array([ref["relres"]]), f"{what}: relres")


def check(kind, inverse):
    """Stops after 1 .. 2 RESTART + 2 steps; F of a 24 x 24 grid (its solves run
    in the LDS of one compute unit) or, inverse, the products with G."""
    if kind == "breakdown":
        for steps in range(1, RESTART + 1):
            A = _bidiagonal(64)
            A.val[A.rowptr[steps]] = 0.0  # the chain ends after `steps` coordinates
            b = np.zeros(A.n)
            b[0] = 1.0
            rp, ci, _, vF, _ = O.ilu(A, 0)
            vF[:] = (ci == np.repeat(np.arange(A.n), np.diff(rp))).astype(np.float64)
            pat = T.symbolic(g(A.rowptr), g(A.col), 0)
            ref = O.gmres(A.n, A.rowptr, A.col, A.val, rp, ci, vF, b, restart=RESTART, maxit=20, rtol=1e-13,
                          inverse=inverse)
            assert ref["iters"] == steps
            x, info = T.gmres(pat, g(A.val), g(vF), g(b), restart=RESTART, maxit=20, rtol=1e-13, inverse=inverse)
            _same(x, info, ref, f"breakdown after {steps} inverse {inverse}")
        return
    A = I.conv_diff_2d(24, 1.0, 5.0, -3.0)
    b = np.random.default_rng(24).standard_normal(A.n)
    rp, ci, _, vF, _ = O.ilu(A, 1)
    m = O.inverse(A.n, rp, ci, vF) if inverse else vF
    args = (A.n, A.rowptr, A.col, A.val, rp, ci, m, b)
    long = O.gmres(*args, restart=RESTART, maxit=2 * RESTART + 2, rtol=1e-14, inverse=inverse)
    assert long["iters"] == 2 * RESTART + 2
    pat = T.symbolic(g(A.rowptr), g(A.col), 1)
    norm = float(np.linalg.norm(b))
    for steps in range(1, 2 * RESTART + 3):
        opt = dict(restart=RESTART, maxit=steps, rtol=1e-14) if kind == "maxit" else dict(
            restart=RESTART, maxit=40, rtol=float(long["hist"][steps - 1]) / norm * (1.0 + 1e-9))
        ref = O.gmres(*args, **opt, inverse=inverse)
        x, info = T.gmres(pat, g(A.val), g(m), g(b), **opt, inverse=inverse)
        _same(x, info, ref, f"{kind} after {steps} inverse {inverse}")
