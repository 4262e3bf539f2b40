"""A row of L~ without entries has x_i = b_i: every bit of b_i, also where that is
a signalling NaN (other than the reserved one), in each shape of the solve."""
import numpy as np
import pytest
import torch

import oracle
from paper_0803_0048_amd import binding as T
from paper_0803_0048_amd import inputs
from tests.gpu_util import bits, g, log

pytestmark = pytest.mark.gpu

SNAN = np.array([0x7FF0000000000001, 0xFFF0000000000123, 0x7FF4000000000000], np.uint64)


@pytest.mark.parametrize("name", ["lds", "lds timed", "chunks", "blocks", "rows", "lanes"])
def test_first_level(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    log(f"[gpu] {name}")
    A, k = {"lds": (inputs.conv_diff_2d(64, 1.0, 3.0, 2.0), 1), "chunks": (inputs.conv_diff_2d(150, 1.0, 3.0, 2.0), 1),
            "blocks": (inputs.random_banded(20000, 5), 2)}.get(name.split()[0], (inputs.random_banded(20000, 5), 0))
    rp, ci, _, vF, _ = oracle.ilu(A, k)
    rows = np.repeat(np.arange(A.n), np.diff(rp))
    first = np.flatnonzero(np.bincount(rows[ci < rows], minlength=A.n) == 0)
    b = np.random.default_rng(3).standard_normal(A.n)
    b.view(np.uint64)[first] = SNAN[np.arange(first.size) % SNAN.size]
    ctx = T.context(0)
    for fn in (ctx.set_grid, ctx.set_solver, ctx.set_numeric, ctx.set_placement, ctx.set_group, ctx.set_tickets):
        fn(0)
    ctx.set_solver({"rows": ctx.SOLVER_DEVICE, "lanes": ctx.SOLVER_LANES}.get(name, 0))
    ctx.set_timing("timed" in name)
    try:
        _, x = T.apply(T.symbolic(g(A.rowptr), g(A.col), k), g(vF), g(b), return_x=True)
    finally:
        ctx.set_solver(0)
        ctx.set_timing(False)
    x_ref, _ = oracle.apply(A.n, rp, ci, vF, b)
    assert np.array_equal(bits(x_ref)[first], b.view(np.uint64)[first])
    assert np.array_equal(bits(x)[first], b.view(np.uint64)[first])
