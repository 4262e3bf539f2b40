"""Race check of the library's own choices, run against the jitter build
(libtpilu_jitter.so, see jitter_check.py) as ``TPILU_LIBRARY=jitter python -m
tests.jitter_check_auto`` in a process of its own (test_gpu_jitter_auto.py).

Cases: GMRES stops at every position of a cycle, the host late to read; the
solves at the smallest limit of the watchdog."""
from __future__ import annotations

import os
import sys

import torch

from paper_0803_0048_amd import binding as T
from tests import gmres_stops
from tests.gpu_util import log
from tests.jitter_check import loaded_jitter_build
from tests.test_gpu_bounded_waits import check_solve


def main() -> int:
    assert os.environ.get("TPILU_LIBRARY") == "jitter", "run with TPILU_LIBRARY=jitter"
    torch.cuda.set_device(0)
    T.load_library()
    assert loaded_jitter_build(), "the jitter build is not the library in use"
    for kind in gmres_stops.KINDS:
        for inverse in (False, True):
            log(f"jitter: GMRES stop {kind} inverse {inverse}")
            gmres_stops.check(kind, inverse)
    for name in ("lds", "chunks", "blocks"):
        log(f"jitter: waits of the solves, {name}")
        check_solve(name)
    log("jitter build: all cases bitwise")
    return 0


if __name__ == "__main__":
    sys.exit(main())
