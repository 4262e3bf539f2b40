"""The longest row that Phase I takes (its columns stand in LDS), and one that
does not fit, which is refused before anything is launched for it."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_0803_0048_amd import binding as T
from tests.gpu_util import g, log
from tests.test_gpu_alloc_fallback import _Capped

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


def test_refused_row_leaves_no_memory():
    """Every allocation of the refused call is given back."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 40353
    log(f"[gpu] a row of {n} entries, allocations counted")
    rp, ci = g(np.concatenate([np.arange(n), [2 * n - 1]]).astype(np.int64)), g(
        np.concatenate([np.arange(n - 1), np.arange(n)]).astype(np.int32))
    lib, bud = T.load_library(), _Capped(1 << 34)
    h, p = C.c_void_p(), C.c_void_p()
    stream = C.c_void_p(torch.cuda.current_stream(0).cuda_stream)
    assert lib.tpilu_ctx_create(0, stream, C.cast(bud.alloc, C.c_void_p), C.cast(bud.free, C.c_void_p), None,
                                C.byref(h)) == T.OK
    before = set(bud.live)
    st = lib.tpilu_symbolic(h, n, ci.numel(), C.c_void_p(rp.data_ptr()), C.c_void_p(ci.data_ptr()), 0, C.byref(p))
    torch.cuda.synchronize()
    left = bud.live - before
    lib.tpilu_ctx_destroy(h)
    assert (st, len(left)) == (T.E_DEVICE, 0)
