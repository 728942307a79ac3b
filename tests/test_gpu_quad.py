"""The square's element kernel at the edges of its range: a few cells, one workgroup and one cell more or less,
flat and tall cells, and every boundary type on every side (each side's line of points runs its own way).

Tolerance of one step: in float64 the repository's 1e-12 for a step; in FP32-mixed the modes carry a rounding of
2^-24 = 6e-8 each from storing, the volume term and the edge term, 1e-6 leaves a factor of five."""
import numpy as np
import pytest

import oracle as O
from paper_1601_08145_amd import inputs as I
from paper_1601_08145_amd import lxw as L
from tests.helpers import rel_l1

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [L.FP64, L.FP32_MIXED])
@pytest.mark.parametrize("nx,ny,height,bc", [
    (2, 2, 1.0, [2, 1, 3, 2]), (16, 16, 1.0, [1, 2, 2, 3]), (5, 51, 40.0, [2, 3, 1, 2]), (257, 2, 0.002, [3, 2, 2, 1]),
    (17, 15, 0.1, [0, 0, 0, 0])])
def test_step(nx, ny, height, bc, precision):
    box = (0.0, 1.0, 0.0, height)
    Q = I.random_modal_state(nx * ny, 2, 9, seed=nx, amp=0.3, rough_frac=0.1, rough_amp=2.0, p_range=(1e-3, 1))
    inflow = [1.2, 0.5, -0.2, 3.0]
    S = L.Solver(L.Mesh.cart(nx, ny, *box, bc), precision=precision, inflow=inflow)
    ref = O.Solver(O.Mesh.cart(nx, ny, *box, bc), inflow=inflow)
    for s in (S, ref):
        s.set_state(Q)
        s.step()
    got, want = S.get_state()[0], ref.get_state()[0]
    assert max(rel_l1(got[:, c], want[:, c]) for c in range(4)) <= (1e-12 if precision == L.FP64 else 1e-6)
