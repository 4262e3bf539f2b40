"""More rows than a launch of sixteen lanes a row has threads for (2^28): the map
from A's entries to F's slots of a two-entry-a-row matrix whose F is A."""
import pytest
import torch

from paper_0803_0048_amd import binding as T
from tests.gpu_util import log

pytestmark = [pytest.mark.gpu, pytest.mark.slow]


def test_map_of_a_into_f():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.mem_get_info()[0] < 150e9:
        pytest.skip("needs 150 GB of device memory")
    n, step = 2 ** 28 + 5, 1 << 20  # row i holds column i - step, if there is one: 257 levels
    log(f"[gpu] {n} rows")
    i = torch.arange(n, device="cuda")
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum((i >= step).long() + 1, 0, out=rp[1:])
    ci = torch.empty(int(rp[-1]), dtype=torch.int32, device="cuda")
    ci[rp[1:] - 1] = i.int()
    ci[rp[:-1][step:]] = (i[step:] - step).int()
    del i
    torch.cuda.empty_cache()
    log("[gpu] symbolic")
    pat = T.symbolic(rp, ci, 0)
    assert (pat.nnz_f, pat.info["depth_l"], pat.info["depth_u"]) == (ci.numel(), 257, 1)
    ex = pat.export()
    assert torch.equal(ex["rowptr"], rp) and torch.equal(ex["col"], ci)
    assert torch.equal(ex["a2f"], torch.arange(ci.numel(), dtype=torch.int32, device="cuda"))
    del pat, ex, rp, ci
    torch.cuda.empty_cache()
