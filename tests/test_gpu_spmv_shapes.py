"""SpMV at the edges of its choice of tile: diagonal matrices, up to three
entries a row with and without a longer one, one row that holds most of the
entries; bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_0803_0048_amd import binding as T
from paper_0803_0048_amd import inputs
from tests.gpu_util import assert_bits_equal, g, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,lens", [
    (1, {}), (63, {}), (64, {}), (65, {}), (4161, {}), (1, {0: 1}), (65, {64: 2}), (200, {0: 64}), (200, {0: 65}),
    (200, {i: 3 for i in range(200)}), (200, {i: 3 + (i == 7) for i in range(200)}), (129, {i: 4 for i in range(129)}),
    (1500, {3: 1023}), (1500, {3: 1024}), (40000, {39999: 1024}), (70000, {5: 1024}), (2000, {i: 9 for i in range(2000)})])
def test_spmv(n, lens):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    log(f"[gpu] n={n}")
    rng = np.random.default_rng(n)
    cols = [np.array([i]) for i in range(n)]
    for i, k in lens.items():
        c = rng.choice(n, size=min(k, n), replace=False)
        cols[i] = np.unique(np.append(c[: min(k, n) - 1], i))
    rowptr = np.zeros(n + 1, np.int64)
    np.cumsum([c.size for c in cols], out=rowptr[1:])
    A = inputs.CSR(n, rowptr, np.concatenate(cols).astype(np.int32), rng.standard_normal(rowptr[-1]))
    b = rng.standard_normal(n)
    b[rng.integers(0, n, 2)] = [np.inf, -0.0]
    pat = T.symbolic(g(A.rowptr), g(A.col), 0)
    assert_bits_equal(T.spmv(pat, g(A.val), g(b)), oracle.spmv(n, A.rowptr, A.col, A.val, b), "spmv")
