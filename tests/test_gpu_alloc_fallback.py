"""Allocations that fail and that the library can do without: the call goes on
with what it gets, whatever error the failed allocation left in the runtime."""
from __future__ import annotations

import ctypes as C

import numpy as np
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

    def __init__(self, cap, but=()):
        self.cap, self.but, self.live, self.refused = cap, but, set(), []
        self.hip = _hip()
        self.alloc, self.free = ALLOC_FN(self._alloc), FREE_FN(self._free)

    def _alloc(self, nbytes, user):
        p = C.c_void_p()
        st = self.hip.hipMalloc(C.byref(p), nbytes if nbytes <= self.cap and nbytes not in self.but else 1 << 50)
        if st != 0 or not p.value:
            self.refused.append(nbytes)
            return None
        self.live.add(p.value)
        return p.value

    def _free(self, p, user):
        self.live.discard(p)
        self.hip.hipFree(p)


def _solve(A, k, bud):
    """Pattern, factor and solve through a context with that allocator, against
    the oracle."""
    rpF, ciF, lvF, vF, _ = O.ilu(A, k)
    lib = T.load_library()
    h, p = C.c_void_p(), C.c_void_p()
    stream = C.c_void_p(torch.cuda.current_stream(0).cuda_stream)
    assert lib.tpilu_ctx_create(0, stream, C.cast(bud.alloc, C.c_void_p), C.cast(bud.free, C.c_void_p), None,
                                C.byref(h)) == T.OK
    rp, ci, av = g(A.rowptr), g(A.col), g(A.val)
    ptr = lambda t: C.c_void_p(t.data_ptr())  # noqa: E731
    try:
        st = lib.tpilu_symbolic(h, A.n, A.nnz, ptr(rp), ptr(ci), k, C.byref(p))
        assert bud.refused, "no request was refused"
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


def _need_gpu(what):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    log(f"[gpu] {what}")


# the shared blocks of Phase I alone (the largest array of this pattern takes 2.2
# MB), and with the plan's 2.9 MB allowed
@pytest.mark.parametrize("cap", [5 << 19, 1 << 22])
def test_phase_one_without_large_blocks(cap):
    _need_gpu(f"allocations of at most {cap} bytes")
    _solve(I.conv_diff_2d(200, 1.0, 3.0, 2.0), 1, _Capped(cap))


@pytest.mark.parametrize("m,band", [(200, 0), (300, 0), (0, 40000)])
def test_without_level_chunks(m, band):
    """The arrays of 16 bytes a row (records, heads and parts of the level
    orders, records of the plan) cannot be had."""
    A = I.conv_diff_2d(m, 1.0, 3.0, 2.0) if m else I.random_banded(band, 5)
    _need_gpu(f"n = {A.n} without level chunks")
    sixteen = (16 * A.n + 255) // 256 * 256
    _solve(A, 1, _Capped((8 if m else 40) * sixteen, {sixteen}))


def test_plan_leaves_memory():
    """With little memory free the plan of Phase II (208 bytes a row here) is not
    laid down; the factor is the same."""
    _need_gpu("plan with 2.5 GB free")
    A = I.conv_diff_3d(100, 1.0, np.ones(3))
    rp, ci, av = g(A.rowptr), g(A.col), g(A.val)
    used, factors = [], []
    torch.cuda.empty_cache()
    for free in (None, 5 << 29):
        rest = torch.empty(torch.cuda.mem_get_info()[0] - free, dtype=torch.uint8, device="cuda") if free else None
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        pat = T.symbolic(rp, ci, 1)
        torch.cuda.synchronize()
        used.append(before - torch.cuda.mem_get_info()[0])
        del rest
        torch.cuda.empty_cache()
        factors.append(T.numeric(pat, av).cpu().numpy().view(np.uint64))
        del pat
    plan = 208 * A.n
    log(f"pattern {used[0]} bytes, {used[1]} with little free")
    assert plan * 0.9 < used[0] - used[1] < plan * 1.2, (used, plan)
    assert np.array_equal(*factors)
