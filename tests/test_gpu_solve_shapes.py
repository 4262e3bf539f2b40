"""The automatic shapes of the single-instance solves at the edges of their
tiles, bit for bit against the oracle: one compute unit with x in LDS, level
chunks on one XCD, blocks of consecutive rows."""
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


def _lower_random(n, half, seed, reach, wide=0):
    """CSR with `half` distinct columns on either side of the diagonal, at most `reach`
    away and (wide) at least `wide` away, so that rows closer together are independent."""
    rng = np.random.default_rng(seed)
    rows, cols = [np.arange(n)], [np.arange(n)]
    for i in range(n):
        for lo, hi in ((max(0, i - reach), i - wide), (i + 1 + wide, min(n, i + reach + 1))):
            if hi > lo:
                c = rng.choice(np.arange(lo, hi), size=min(half, hi - lo), replace=False)
                rows.append(np.full(c.size, i))
                cols.append(c)
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    order = np.lexsort((cols, rows))
    rows, cols = rows[order], cols[order]
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(rows, minlength=n), out=rowptr[1:])
    val = rng.uniform(-1.0, 1.0, size=cols.size)
    val[rows == cols] = 1.1 * (2 * half + 1)
    return inputs.CSR(n, rowptr, cols.astype(np.int32), val)


def _check(A, k, b, edit=None):
    dev = torch.device("cuda")
    rp, ci, _, vF, _ = oracle.ilu(A, k)
    if edit is not None:
        edit(rp, ci, vF)
    pat = T.symbolic(torch.from_numpy(A.rowptr).to(dev), torch.from_numpy(A.col).to(dev), k)
    f, bt = torch.from_numpy(vF).to(dev), torch.from_numpy(b).to(dev)
    x_ref, y_ref = oracle.apply(A.n, rp, ci, vF, b)
    y, x = T.apply(pat, f, bt, return_x=True)
    assert_bits_equal(x, x_ref, "x")
    assert_bits_equal(y, y_ref, "y")
    # without x, twice in a row, and with the sweeps timed apart
    y2 = torch.empty_like(bt)
    for timing in (False, False, True):
        T.context().set_timing(timing)
        try:
            T.apply(pat, f, bt, out=y2)
            assert_bits_equal(y2, y_ref, f"y, timing {timing}")
        finally:
            T.context().set_timing(False)
            for kind in range(3):
                T.context().read_timing(kind)
    return pat


@pytest.mark.parametrize("n,half,reach,wide", [
    (1, 1, 1, 0), (2, 1, 1, 0), (63, 2, 9, 0), (64, 4, 40, 0), (65, 5, 64, 0), (130, 8, 100, 0), (200, 9, 60, 0),
    (1025, 16, 300, 0), (1500, 17, 300, 0), (3000, 3, 2999, 1100), (16383, 1, 40, 0), (16384, 1, 40, 0),
    (16385, 1, 40, 0)])
def test_small_systems(n, half, reach, wide):
    """One compute unit: row halves of 1 to 16 entries and one more, levels of one chunk and of
    many, the largest system that fits and one more row."""
    A = _lower_random(n, half, 11 + n, reach, wide)
    _check(A, 0, np.random.default_rng(n).standard_normal(n))


@pytest.mark.parametrize("n,half", [(4096, 2), (4097, 4), (4100, 5), (6000, 8), (5000, 9), (20000, 16), (20001, 3),
                                    (20000, 17), (20000, 33)])
def test_level_chunks(n, half):
    """Few, wide levels: chunks of 64 positions, whole and partial, of every entry width
    and of rows taken in two and three rounds."""
    A = _lower_random(n, half, 5 + n, n - 1, n // 9)
    _check(A, 0, np.random.default_rng(n).standard_normal(n))


@pytest.mark.parametrize("n,k", [(64, 1), (65, 2), (127, 2), (700, 2), (1984, 1), (1985, 1), (2049, 2)])
def test_blocks(n, k):
    """Random banded matrices: whole and partial last blocks, windows at both ends of the
    matrix, windows too full for the block kernel (small n at k = 2)."""
    A = inputs.random_banded(n, 3, band=min(n // 2, 300 + n // 2))
    _check(A, k, np.random.default_rng(n).standard_normal(n))


def test_blocks_nothing_in_window():
    """Rows whose dependencies are all far away, and rows with none."""
    A = _lower_random(3000, 20, 9, 900, 260)
    _check(A, 0, np.random.default_rng(1).standard_normal(A.n))


@pytest.mark.parametrize("shape", ["lds", "chunks", "blocks"])
def test_special_values(shape):
    """Infinities, NaN, zeros of both signs and subnormals in the factor and the right-hand side."""
    A = {"lds": lambda: _lower_random(300, 3, 1, 60, 0), "chunks": lambda: _lower_random(5000, 3, 1, 4999, 600),
         "blocks": lambda: inputs.random_banded(1500, 3, band=700)}[shape]()
    rng = np.random.default_rng(2)
    b = rng.standard_normal(A.n)
    b[rng.integers(0, A.n, 40)] = -0.0
    b[rng.integers(A.n // 2, A.n, 3)] = [np.inf, np.nan, 5e-324]

    def edit(rp, ci, vF):
        off = np.flatnonzero(ci != np.repeat(np.arange(A.n), np.diff(rp)))
        at = rng.permutation(off)[:60]
        vF[at[:40]] = np.where(rng.random(40) < 0.5, 0.0, -0.0)
        vF[at[40:44]] = [np.inf, -np.inf, np.nan, 1e308]

    _check(A, 0 if shape != "blocks" else 1, b, edit)
    # all of it zero, both signs: the result's zeros keep their signs
    _check(A, 0 if shape != "blocks" else 1, np.where(rng.random(A.n) < 0.5, 0.0, -0.0))
    # the reserved pattern in the right-hand side is reported and becomes a NaN
    dev = torch.device("cuda")
    pat = T.symbolic(torch.from_numpy(A.rowptr).to(dev), torch.from_numpy(A.col).to(dev), 0)
    f = T.numeric(pat, torch.from_numpy(A.val).to(dev))
    bad = torch.ones(A.n, dtype=torch.float64, device=dev)
    bad.view(torch.int64)[A.n // 3] = 0x7FF4A5A5A5A5A5A5
    y, x = T.apply(pat, f, bad, return_x=True)
    with pytest.raises(T.TpiluError):
        T.check(pat)
    assert torch.isnan(x[A.n // 3])
    T.apply(pat, f, torch.ones_like(bad))
    T.check(pat)


@pytest.mark.parametrize("n,k", [(64, 1), (700, 2), (1984, 1), (1985, 2), (4097, 2), (20000, 1)])
def test_levels_by_blocks(n, k):
    """The depths that the blocks of 64 rows find are those of a sequential walk."""
    A = inputs.random_banded(n, 3, band=min(n // 2, 300 + n // 2))
    rp, ci, _, _, _ = oracle.ilu(A, k)
    lo, up = np.zeros(n, np.int64), np.zeros(n, np.int64)
    for i in range(n):
        c = ci[rp[i]:rp[i + 1]]
        lo[i] = 1 + max(lo[c[c < i]], default=0)
    for i in range(n - 1, -1, -1):
        c = ci[rp[i]:rp[i + 1]]
        up[i] = 1 + max(up[c[c > i]], default=0)
    dev = torch.device("cuda")
    info = T.symbolic(torch.from_numpy(A.rowptr).to(dev), torch.from_numpy(A.col).to(dev), k).info
    assert (info["depth_l"], info["depth_u"]) == (lo.max(), up.max())
