"""GMRES stops (tolerance, maxit, breakdown) at every position of a cycle with
the next step launched ahead, bit for bit against the oracle."""
import pytest
import torch

from tests import gmres_stops
from tests.gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inverse", [False, True])
@pytest.mark.parametrize("kind", gmres_stops.KINDS)
def test_stop(kind, inverse):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    log(f"[gpu] gmres stop {kind} inverse {inverse}")
    gmres_stops.check(kind, inverse)
    torch.cuda.synchronize()
