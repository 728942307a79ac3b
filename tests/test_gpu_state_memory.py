"""State transfer takes no device memory of its own."""
import numpy as np
import pytest

import torch

from paper_1601_08145_amd import lxw as L
from tests.test_gpu_state import state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [L.FP64, L.FP32_MIXED])
def test_transfer_needs_no_device_memory(precision):
    """A solver's memory is allocated when it is made: states in host memory (here 22 and 37 MB) are set and read
    with the device's free memory as it is."""
    def rounds(n, cells):
        line = L.Mesh.line(n, 0.0, 1.0, 1, 1)
        quads = [L.Mesh.cart(c, c, 0.0, 1.0, 0.0, 1.0, [1, 1, 1, 1]) for c in cells]
        S, B = L.Solver(line, precision=precision), L.Batch(quads, precision=precision)
        Q = state(line, 2, 1, precision == L.FP32_MIXED)
        Qs = [state(m, 2, 2, precision == L.FP32_MIXED) for m in quads]
        torch.cuda.synchronize()
        free = [torch.cuda.mem_get_info()[0]]
        S.get_state()
        free.append(torch.cuda.mem_get_info()[0])
        S.set_state(Q)
        for b in (0, 1):
            B.set_state(b, Qs[b])
        free.append(torch.cuda.mem_get_info()[0])
        assert np.array_equal(S.get_state()[0], Q)
        for b in (0, 1):
            assert np.array_equal(B.get_state(b)[0], Qs[b])
        free.append(torch.cuda.mem_get_info()[0])
        return free

    rounds(100, (4, 8))  # what the first calls of a process load
    free = rounds(300_000, (80, 360))
    assert free == free[:1] * 4
