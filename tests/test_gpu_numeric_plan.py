"""Phase II with several rows per wavefront at the edges of its shapes, bit for
bit against the oracle: rows that just fill 8, 16, 32 and 64 lanes and one entry
more, U~ that just fits in LDS and one entry more, narrow and wide levels."""
import numpy as np
import pytest
import torch

import oracle
from paper_0803_0048_amd import binding as T
from paper_0803_0048_amd import inputs

from tests.gpu_util import assert_bits_equal, log

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu_guard(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    log(f"[gpu] {request.node.nodeid}")
    yield
    torch.cuda.synchronize()


def _band(n, lower, upper, seed):
    """A full band of `lower` and `upper` columns either side of the diagonal."""
    rng = np.random.default_rng(seed)
    i = np.arange(n)
    cols = i[:, None] + np.arange(-lower, upper + 1)[None, :]
    ok = (cols >= 0) & (cols < n)
    rowptr = np.concatenate([[0], np.cumsum(ok.sum(1))]).astype(np.int64)
    col = cols[ok].astype(np.int32)
    val = rng.uniform(-1.0, 1.0, col.size)
    val[col == np.repeat(i, ok.sum(1))] = 1.1 * (lower + upper + 1)
    return inputs.CSR(n, rowptr, col, val)


def _check(A, k, edit=None, plain_only=False):
    dev = torch.device("cuda")
    val = A.val.copy()
    if edit is not None:
        edit(val)
    pat = T.symbolic(torch.from_numpy(A.rowptr).to(dev), torch.from_numpy(A.col).to(dev), k)
    a = torch.from_numpy(val).to(dev)
    rp, ci, _ = oracle.symbolic(A.n, A.rowptr, A.col, k)
    for fused in (False, True) if not plain_only else (False,):
        ref = oracle.numeric(A.n, A.rowptr, A.col, val, rp, ci, fused=fused)
        ref = ref[0] if isinstance(ref, tuple) else ref
        T.context().set_fused(fused)
        try:
            f = T.numeric(pat, a)
            assert_bits_equal(f, ref, f"fused {fused}")
            T.numeric(pat, a, out=f)
            assert_bits_equal(f, ref, f"fused {fused}, again")
        finally:
            T.context().set_fused(False)
    return pat


@pytest.mark.parametrize("n,lower,upper", [
    (1, 0, 0), (2, 1, 1), (9, 3, 4), (200, 4, 3), (200, 4, 4), (200, 5, 2), (70, 8, 7), (300, 7, 8), (300, 8, 8),
    (300, 9, 2), (300, 15, 16), (300, 16, 15), (300, 16, 16), (300, 17, 3), (150, 31, 32), (150, 32, 31), (150, 32, 32),
    (150, 33, 2), (9728, 1, 1), (9729, 1, 1)])
def test_full_bands(n, lower, upper):
    """Every row waits on the one before; lanes and pivots of a row used up, and one more."""
    _check(_band(n, lower, upper, n + lower), 0)


@pytest.mark.parametrize("shape,m,k", [
    ("2d", 17, 1), ("2d", 68, 1), ("2d", 90, 2), ("2d", 40, 3), ("7pt", 9, 1), ("7pt", 20, 2), ("7pt", 44, 0),
    ("27pt", 9, 0), ("27pt", 8, 1), ("27pt", 24, 1)])
def test_stencils(shape, m, k):
    """Levels of one part and of many, on one XCD and across the device."""
    A = {"2d": lambda: inputs.conv_diff_2d(m, 1.0, 1.0, 2.0), "7pt": lambda: inputs.conv_diff_3d(m, 1.0, np.ones(3)),
         "27pt": lambda: inputs.stencil27_3d(m, 1.0, np.ones(3))}[shape]()
    _check(A, k)


def test_wide_random():
    A = inputs.random_uniform(20000, 60000, 5)
    _check(A, 0)
    _check(A, 1)


@pytest.mark.parametrize("m", [12, 100])
def test_special_values(m):
    """Zeros of both signs, subnormals, infinities and NaN in A, in LDS and across compute units."""
    A = inputs.conv_diff_2d(m, 1.0, 1.0, 2.0)
    rng = np.random.default_rng(m)
    off = np.flatnonzero(A.col != np.repeat(np.arange(A.n), np.diff(A.rowptr)))

    def edit(val):
        at = rng.permutation(off)[:60]
        val[at[:40]] = np.where(rng.random(40) < 0.5, 0.0, -0.0)
        val[at[40:50]] = 5e-324
        val[at[50:53]] = [np.inf, -np.inf, np.nan]

    _check(A, 1, edit, plain_only=True)


@pytest.mark.parametrize("m,row", [(12, 0), (12, 100), (100, 7777)])
def test_zero_pivot_is_reported(m, row):
    A = inputs.conv_diff_2d(m, 1.0, 1.0, 2.0)
    val = A.val.copy()
    val[(np.repeat(np.arange(A.n), np.diff(A.rowptr)) == row)] = 0.0
    dev = torch.device("cuda")
    pat = T.symbolic(torch.from_numpy(A.rowptr).to(dev), torch.from_numpy(A.col).to(dev), 1)
    with pytest.raises(T.TpiluError) as e:
        T.numeric(pat, torch.from_numpy(val).to(dev))
    assert e.value.bad_row == row


@pytest.mark.parametrize("n,lower,upper,B", [
    (1, 0, 0, 2), (3, 1, 1, 65), (150, 4, 3, 2), (150, 4, 4, 63), (150, 3, 8, 64), (150, 4, 7, 65), (150, 4, 8, 66),
    (120, 5, 6, 7), (120, 8, 7, 130), (90, 8, 8, 3), (60, 9, 2, 5)])
def test_batches(n, lower, upper, B):
    """Instances as lanes: rows that just fill 8, 12 and 16 entries and one more, part and
    whole groups of instances, the forward substitution fused into the factorization or not."""
    A = _band(n, lower, upper, n + lower)
    rng = np.random.default_rng(B)
    val = A.val[:, None] * rng.uniform(0.5, 1.5, (1, B))
    b = rng.standard_normal((n, B))
    dev = torch.device("cuda")
    pat = T.symbolic(torch.from_numpy(A.rowptr).to(dev), torch.from_numpy(A.col).to(dev), 0)
    a, bt = torch.from_numpy(val).to(dev), torch.from_numpy(b).to(dev)
    rp, ci, _ = oracle.symbolic(n, A.rowptr, A.col, 0)
    graph = T.BatchedGraph(pat, a, bt)
    graph.launch()
    torch.cuda.synchronize()
    for fused in (False, True):
        ref = np.stack([oracle.numeric(n, A.rowptr, A.col, val[:, q], rp, ci, fused=fused)[0] for q in range(B)], 1)
        T.context().set_fused(fused)
        try:
            assert_bits_equal(T.numeric(pat, a), ref, f"fused {fused}")
        finally:
            T.context().set_fused(False)
        if not fused:
            y = np.stack([oracle.apply(n, rp, ci, ref[:, q], b[:, q])[1] for q in range(B)], 1)
            assert_bits_equal(graph.f_val, ref, "graph factor")
            assert_bits_equal(graph.y, y, "graph y")
