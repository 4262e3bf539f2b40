"""The watchdog in the dependency levels (Phase I and the transposes of the
adjoint): a wait that runs out ends with TPILU_E_TIMEOUT, everything queued
behind it stays in bounds, and the next call is right again.  The limit is the
smallest there is (1 us), so which waits run out depends on the time a level
takes: a call either reports the time-out or has the oracle's pattern."""
import numpy as np
import pytest
import torch

import oracle
from paper_0803_0048_amd import binding as T
from paper_0803_0048_amd import inputs
from tests.gpu_util import check_pattern, g, log

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu_guard(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    log(f"[gpu] {request.node.nodeid}")
    ctx = T.context(0)
    ctx.set_watchdog(0, -1)
    ctx.set_placement(0)
    yield
    ctx.set_watchdog(0, -1)
    ctx.set_placement(0)
    torch.cuda.synchronize()


def _system(kind):
    if kind == "lanes":  # a lane per node
        return inputs.conv_diff_2d(400, 1.0, 3.0, 2.0), 1, 0
    if kind == "lanes 27":
        return inputs.stencil27_3d(24, 1.0, np.ones(3)), 1, 0
    if kind == "blocks":  # blocks of 64 nodes on one XCD
        return inputs.random_banded(20000, 5), 2, 0
    return inputs.random_banded(20000, 5), 2, T.Context.PLACE_DEVICE  # a wavefront per node


@pytest.mark.parametrize("kind", ["lanes", "lanes 27", "blocks", "wavefronts"])
def test_phase_one(kind):
    A, k, place = _system(kind)
    ctx = T.context(0)
    ctx.set_placement(place)
    ref = oracle.symbolic(A.n, A.rowptr, A.col, k)
    rp, ci = g(A.rowptr), g(A.col)
    ran_out = 0
    for limit in (1, 1, 0):
        ctx.set_watchdog(limit, -1)
        try:
            check_pattern(T.symbolic(rp, ci, k), *ref, A)
        except T.TpiluError as e:
            assert limit and e.status == T.E_TIMEOUT, e
            ran_out += 1
    if kind == "lanes":
        assert ran_out == 2, "waits of about a millisecond without news"


def test_transposes():
    A, k, _ = _system("lanes")
    pat = T.symbolic(g(A.rowptr), g(A.col), k)
    f = T.numeric(pat, g(A.val))
    b = torch.ones(A.n, dtype=torch.float64, device="cuda")
    y, x = T.apply(pat, f, b, return_x=True)
    ctx = T.context(0)
    ctx.set_watchdog(1, -1)
    with pytest.raises(T.TpiluError) as e:
        T.apply_adjoint(pat, f, x, y, b)
    assert e.value.status == T.E_TIMEOUT
    ctx.set_watchdog(0, -1)
    bbar, fbar = T.apply_adjoint(pat, f, x, y, b)
    want = oracle.apply_adjoint(A.n, *(t.cpu().numpy() for t in (pat.export()["rowptr"], pat.export()["col"], f)),
                                x.cpu().numpy(), y.cpu().numpy(), b.cpu().numpy())
    assert np.array_equal(bbar.cpu().numpy(), want[0]) and np.array_equal(fbar.cpu().numpy(), want[1])
