"""The check of a caller's state at the border of p_bar > 0, as separately rounded float64 operations decide it:
p_bar = (gamma - 1) (E - (M.M / 2) / rho) with every product and every sum rounded."""
import numpy as np
import pytest

import torch

from paper_1601_08145_amd import inputs as I
from paper_1601_08145_amd import lxw as L

pytestmark = pytest.mark.gpu


def averages(dim, want, n, seed=1):
    """n averages (rho, M, E) within an ulp of zero pressure whose sign is `want` (1: p > 0, accepted; 0:
    p <= 0, refused) by separately rounded operations, and the opposite where the sum of squares is fused
    (exactly rounded once per term: M_d^2 + k with a single rounding)."""
    from fractions import Fraction as F
    g = np.random.default_rng(seed)
    out = []
    while len(out) < n:
        rho = g.uniform(0.5, 2.0)
        m = g.uniform(-3.0, 3.0, dim)
        sep = fused = 0.0
        for x in m:
            sep = sep + x * x
            fused = float(F(float(x)) * F(float(x)) + F(fused))
        if sep == fused:
            continue
        e = 0.5 * sep / rho
        for E in (np.nextafter(e, 0.0), e, np.nextafter(e, 9.0)):
            p = 0.4 * (E - 0.5 * sep / rho)
            pf = 0.4 * (E - 0.5 * fused / rho)
            if (p > 0.0) == bool(want) and (pf > 0.0) != bool(want):
                out.append([rho, *m, E])
                break
    return np.array(out)


def mesh_of(dim):
    if dim == 3:
        return L.Mesh.tet(*I.lattice_tets(4, 0))
    return L.Mesh.cart(9, 7, 0.0, 1.0, 0.0, 1.0, [1, 1, 1, 1])


@pytest.mark.parametrize("device", [False, True])
@pytest.mark.parametrize("dim", [2, 3])
def test_border(dim, device):
    mesh = mesh_of(dim)
    S = L.Solver(mesh, gamma=1.4)
    give = (lambda q: torch.from_numpy(q).cuda()) if device else (lambda q: q)
    Q = np.zeros(S.shape)
    Q[:, :, 0] = averages(dim, 1, mesh.N)
    S.set_state(give(Q))  # every one accepted
    assert np.array_equal(S.get_state()[0], Q)
    refused = averages(dim, 0, 8)
    for c, q in enumerate(refused):
        bad = Q.copy()
        bad[3 + c, :, 0] = q
        with pytest.raises(L.LxwError, match=f"element {3 + c}\\)") as e:
            S.set_state(give(bad))
        assert e.value.name == "LXW_ERR_STATE"
