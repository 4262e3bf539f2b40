"""Row sums in tiles (SpMV and the products with the incomplete inverses) at the
edges of their tiles: empty halves, rows one entry shorter and longer than a
tile and a wavefront's rows, one long row among short ones."""
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


@pytest.mark.parametrize("n,lens", [
    (1, (1,)), (15, (1,)), (17, (2, 3)), (63, (7, 8, 9)), (65, (8,)), (129, (15, 16, 17)), (300, (31, 32, 33)),
    (1000, (1, 1, 1, 1, 65)), (257, (64,)), (2000, (1, 40, 2, 33, 500))])
def test_row_products(n, lens):
    rng = np.random.default_rng(n)
    cols = []
    for i in range(n):
        k = min(n, lens[i % len(lens)])
        c = rng.choice(n, size=k, replace=False)
        cols.append(np.unique(np.append(c[: max(0, k - 1)], i)))
    rowptr = np.zeros(n + 1, np.int64)
    np.cumsum([c.size for c in cols], out=rowptr[1:])
    A = inputs.CSR(n, rowptr, np.concatenate(cols).astype(np.int32), rng.standard_normal(rowptr[-1]))
    b = rng.standard_normal(n)
    dev = torch.device("cuda")
    g = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    rp, ci = oracle.symbolic(n, A.rowptr, A.col, 0)[:2]
    pat = T.symbolic(g(A.rowptr), g(A.col), 0)
    assert_bits_equal(T.spmv(pat, g(A.val), g(b)), oracle.spmv(n, A.rowptr, A.col, A.val, b), "spmv")
    G = rng.standard_normal(ci.size)
    assert_bits_equal(T.apply_inverse(pat, g(G), g(b)), oracle.apply_inverse(n, rp, ci, G, b)[1], "products")
