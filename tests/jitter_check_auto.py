"""Race check of the library's own choices, run against the jitter build
(libtpilu_jitter.so, see jitter_check.py) as ``TPILU_LIBRARY=jitter python -m
tests.jitter_check_auto`` in a process of its own (test_gpu_jitter_auto.py).

Cases: GMRES stops at every position of a cycle, the host late to read; the
solves at the smallest limit of the watchdog; pattern, factorization (either
rounding of the update), both substitutions and a batch of systems whose shapes
the library picks: one compute unit's LDS, several rows per wavefront on one XCD
and across the device with 8 and 64 lanes a row, level chunks, blocks of rows."""
from __future__ import annotations

import os
import sys

import numpy as np
import torch

import oracle as O
from paper_0803_0048_amd import binding as T
from paper_0803_0048_amd import inputs as I
from tests import gmres_stops
from tests.gpu_util import assert_bits_equal, check_pattern, g, log
from tests.jitter_check import batched, loaded_jitter_build
from tests.test_gpu_bounded_waits import check_solve


def automatic(name, A, k):
    log(f"jitter: {name} n={A.n} k={k}, automatic choices")
    ctx = T.context(0)
    rpF, ciF, lvF = O.symbolic(A.n, A.rowptr, A.col, k)
    b = np.random.default_rng(A.n).standard_normal(A.n)
    pat = T.symbolic(g(A.rowptr), g(A.col), k)
    check_pattern(pat, rpF, ciF, lvF, A)
    for fused in (True, False):
        vF, _ = O.numeric(A.n, A.rowptr, A.col, A.val, rpF, ciF, fused=fused)
        ctx.set_fused(fused)
        try:
            f = T.numeric(pat, g(A.val))
        finally:
            ctx.set_fused(False)
        assert_bits_equal(f, vF, f"{name} F fused {fused}")
    x_ref, y_ref = O.apply(A.n, rpF, ciF, vF, b)
    y, x = T.apply(pat, f, g(b), return_x=True)
    assert_bits_equal(x, x_ref, f"{name} x")
    assert_bits_equal(y, y_ref, f"{name} y")
    assert_bits_equal(T.apply(pat, f, g(b)), y_ref, f"{name} y without x")


def main() -> int:
    assert os.environ.get("TPILU_LIBRARY") == "jitter", "run with TPILU_LIBRARY=jitter"
    torch.cuda.set_device(0)
    T.load_library()
    assert loaded_jitter_build(), "the jitter build is not the library in use"
    one = np.ones(3)
    automatic("2-D 64^2", I.conv_diff_2d(64, 1.0, 1.0, 2.0), 1)
    automatic("2-D 150^2", I.conv_diff_2d(150, 1.0, 1.0, 2.0), 1)
    automatic("7-point 44^3", I.conv_diff_3d(44, 1.0, one), 0)
    automatic("7-point 28^3", I.conv_diff_3d(28, 1.0, one), 2)
    automatic("27-point 12^3", I.stencil27_3d(12, 1.0, one), 1)
    automatic("27-point 24^3", I.stencil27_3d(24, 1.0, one), 1)
    automatic("random banded", I.random_banded(6000, 1002), 2)
    c = I.batched_conv_diff_2d_ilu2(B=70, m=24)
    for k in (0, 1, 2):
        batched(f"batched 2-D 24^2 ILU({k})", c["A"], k, c["b"])
    for kind in gmres_stops.KINDS:
        for inverse in (False, True):
            log(f"jitter: GMRES stop {kind} inverse {inverse}")
            gmres_stops.check(kind, inverse)
    for name in ("lds", "chunks", "blocks"):
        log(f"jitter: waits of the solves, {name}")
        check_solve(name)
    log("jitter build: all cases bitwise")
    return 0


if __name__ == "__main__":
    sys.exit(main())
