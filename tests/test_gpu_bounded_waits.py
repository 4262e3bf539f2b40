"""The kernels that the library chooses by itself under the watchdog: the
factorization of a small system with a row that is never published, and the
solves at the smallest limit there is, where a call either reports the time-out
or has the oracle's bits; the call after it is right again."""
import numpy as np
import pytest
import torch

import oracle
from paper_0803_0048_amd import binding as T
from paper_0803_0048_amd import inputs
from tests.gpu_util import assert_bits_equal, g, log

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu_guard(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    log(f"[gpu] {request.node.nodeid}")
    ctx = T.context(0)
    for fn in (ctx.set_grid, ctx.set_solver, ctx.set_numeric, ctx.set_placement, ctx.set_group, ctx.set_tickets):
        fn(0)
    ctx.set_watchdog(0, -1)
    yield
    ctx.set_watchdog(0, -1)
    torch.cuda.synchronize()


@pytest.mark.parametrize("k,fused", [(0, False), (1, False), (1, True)])
def test_small_factorization(k, fused):
    A = inputs.conv_diff_2d(40, 1.0, 3.0, 2.0)
    rp, ci, _ = oracle.symbolic(A.n, A.rowptr, A.col, k)
    vF, _ = oracle.numeric(A.n, A.rowptr, A.col, A.val, rp, ci, fused=fused)
    pat = T.symbolic(g(A.rowptr), g(A.col), k)
    ctx = T.context(0)
    ctx.set_fused(fused)
    try:
        ctx.set_watchdog(20000, 100)
        with pytest.raises(T.TpiluError) as e:
            T.numeric(pat, g(A.val))
        assert e.value.status == T.E_TIMEOUT
        ctx.set_watchdog(0, -1)
        assert_bits_equal(T.numeric(pat, g(A.val)), vF, "F")
    finally:
        ctx.set_fused(False)


def systems():
    """Both sweeps in the LDS of one compute unit; by level chunks; by blocks."""
    return {"lds": (inputs.conv_diff_2d(64, 1.0, 3.0, 2.0), 1), "chunks": (inputs.conv_diff_2d(150, 1.0, 3.0, 2.0), 1),
            "blocks": (inputs.random_banded(20000, 5), 2)}


def check_solve(name):
    """Whether the solve at the smallest limit ran out."""
    A, k = systems()[name]
    rp, ci, _, vF, _ = oracle.ilu(A, k)
    b = np.random.default_rng(7).standard_normal(A.n)
    pat = T.symbolic(g(A.rowptr), g(A.col), k)
    f, ctx = g(vF), T.context(0)
    y_ref = oracle.apply(A.n, rp, ci, vF, b)[1]
    ctx.set_watchdog(1, -1)
    y = T.apply(pat, f, g(b))
    ran_out = False
    try:
        T.check(pat)
        assert_bits_equal(y, y_ref, f"{name} y at the smallest limit")
    except T.TpiluError as e:
        assert e.status == T.E_TIMEOUT
        ran_out = True
    ctx.set_watchdog(0, -1)
    y = T.apply(pat, f, g(b))
    T.check(pat)
    assert_bits_equal(y, y_ref, f"{name} y")
    return ran_out


@pytest.mark.parametrize("name", ["lds", "chunks", "blocks"])
def test_solve(name):
    log(f"ran out: {check_solve(name)}")
