"""Allocations that fail and that the library can do without: the call goes on
with what it gets, whatever error the failed allocation left in the runtime."""
from __future__ import annotations

import ctypes as C

import pytest
import torch

import oracle as O
from paper_0803_0048_amd import binding as T
from paper_0803_0048_amd import inputs as I
from tests.gpu_util import assert_bits_equal, g, log

pytestmark = pytest.mark.gpu

ALLOC_FN = C.CFUNCTYPE(C.c_void_p, C.c_size_t, C.c_void_p)
FREE_FN = C.CFUNCTYPE(None, C.c_void_p, C.c_void_p)


def _hip():
    with open("/proc/self/maps") as fh:
        path = next(ln.split()[-1] for ln in fh if "libamdhip64" in ln)
    hip = C.CDLL(path)
    hip.hipMalloc.argtypes = [C.POINTER(C.c_void_p), C.c_size_t]
    hip.hipFree.argtypes = [C.c_void_p]
    return hip


class _Capped:
    """hipMalloc up to `cap` bytes a request; a larger one fails as hipMalloc does
    when memory is short, its error left behind.  (Only calls that cannot raise:
    a callback that raises leaves its result undefined.)"""

    def __init__(self, cap):
        self.cap, self.live, self.refused = cap, set(), []
        self.hip = _hip()
        self.alloc, self.free = ALLOC_FN(self._alloc), FREE_FN(self._free)

    def _alloc(self, nbytes, user):
        p = C.c_void_p()
        st = self.hip.hipMalloc(C.byref(p), nbytes if nbytes <= self.cap else 1 << 50)
        if st != 0 or not p.value:
            self.refused.append(nbytes)
            return None
        self.live.add(p.value)
        return p.value

    def _free(self, p, user):
        self.live.discard(p)
        self.hip.hipFree(p)


# the shared blocks of Phase I alone (the largest array of this pattern takes 2.2
# MB), and with the plan's 3.6 MB allowed
@pytest.mark.parametrize("cap", [5 << 19, 1 << 22])
def test_phase_one_without_large_blocks(cap):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    log(f"[gpu] allocations of at most {cap} bytes")
    A, k = I.conv_diff_2d(200, 1.0, 3.0, 2.0), 1
    rpF, ciF, lvF, vF, _ = O.ilu(A, k)
    lib = T.load_library()
    bud, h, p = _Capped(cap), C.c_void_p(), C.c_void_p()
    stream = C.c_void_p(torch.cuda.current_stream(0).cuda_stream)
    assert lib.tpilu_ctx_create(0, stream, C.cast(bud.alloc, C.c_void_p), C.cast(bud.free, C.c_void_p), None,
                                C.byref(h)) == T.OK
    rp, ci, av = g(A.rowptr), g(A.col), g(A.val)
    ptr = lambda t: C.c_void_p(t.data_ptr())  # noqa: E731
    try:
        st = lib.tpilu_symbolic(h, A.n, A.nnz, ptr(rp), ptr(ci), k, C.byref(p))
        assert bud.refused, "no request was large enough"
        assert st == T.OK, (st, lib.tpilu_last_error(h), bud.refused)
        f = torch.empty(vF.size, dtype=torch.float64, device="cuda")
        bad = C.c_int64(-1)
        assert lib.tpilu_numeric(h, p, ptr(av), 1, ptr(f), C.byref(bad)) == T.OK
        assert_bits_equal(f, vF, "F")
        b = torch.ones(A.n, dtype=torch.float64, device="cuda")
        y = torch.empty_like(b)
        assert lib.tpilu_apply(h, p, ptr(f), 1, ptr(b), ptr(y), None) == T.OK
        torch.cuda.synchronize()
        assert_bits_equal(y, O.apply(A.n, rpF, ciF, vF, b.cpu().numpy())[1], "y")
        lib.tpilu_pattern_destroy(p)
        assert not bud.live
    finally:
        torch.cuda.synchronize()
        lib.tpilu_ctx_destroy(h)
