"""The longest row that Phase I takes (its columns stand in LDS), and one that
does not fit, which is refused before anything is launched for it."""
import numpy as np
import pytest
import torch

from paper_0803_0048_amd import binding as T
from tests.gpu_util import g, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,fits", [(40352, True), (40353, False)])
def test_longest_row(n, fits):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    log(f"[gpu] a row of {n} entries")
    rp = np.concatenate([np.arange(n), [2 * n - 1]]).astype(np.int64)  # a diagonal and a full last row
    ci = np.concatenate([np.arange(n - 1), np.arange(n)]).astype(np.int32)
    if fits:
        pat = T.symbolic(g(rp), g(ci), 0)
        assert (pat.nnz_f, pat.info["max_row"], pat.info["depth_l"]) == (ci.size, n, 2)
    else:
        with pytest.raises(T.TpiluError) as e:
            T.symbolic(g(rp), g(ci), 0)
        assert e.value.status == T.E_DEVICE
