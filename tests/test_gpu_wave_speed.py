"""Wave speeds beyond float64's range: a cell whose gamma p / rho or |u|^2 overflows is reported, by its number,
in the step that meets it, and never left out of the global wave speed."""
import numpy as np
import pytest

from paper_1601_08145_amd import inputs as I
from paper_1601_08145_amd import lxw as L

pytestmark = pytest.mark.gpu


def case(kind):
    if kind == "line":  # one workgroup, and as separate launches
        return L.Mesh.line(100, 0.0, 1.0, 1, 1), 2
    if kind == "line3":
        return L.Mesh.line(700, 0.0, 1.0, 1, 1), 3
    if kind == "quad":
        return L.Mesh.cart(12, 9, 0.0, 1.0, 0.0, 1.0, [1, 1, 1, 1]), 2
    if kind == "tet":
        return L.Mesh.tet(*I.lattice_tets(4, 0)), 2
    return L.Mesh.tri(*I.lattice_delaunay(14, 0)), 3 if kind == "tri3" else 2


@pytest.mark.parametrize("what", ["pressure", "velocity"])
@pytest.mark.parametrize("speed", [L.SPEED_POINTS, L.SPEED_AVERAGES])
@pytest.mark.parametrize("precision", [L.FP64, L.FP32_MIXED])
@pytest.mark.parametrize("kind", ["line", "line3", "quad", "tri", "tri3", "tet"])
def test_infinite_speed_is_reported(kind, precision, speed, what):
    mesh, degree = case(kind)
    S = L.Solver(mesh, degree=degree, precision=precision, wave_speed=speed)
    Q = I.random_modal_state(mesh.N, mesh.dim, L.n_modes(mesh.kind, degree), seed=2, amp=0.0)
    cell = mesh.N // 3
    Q[cell] = 0.0
    rho = 1e-10
    Q[cell, 0, 0] = rho
    if what == "pressure":  # gamma p / rho = 5.6e309
        Q[cell, -1, 0] = 1e300
    else:  # |u|^2 = 1e310, p / rho far below it: 4e305
        Q[cell, 1, 0] = rho * 1e155
        Q[cell, -1, 0] = 0.5 * (Q[cell, 1, 0] * (Q[cell, 1, 0] / rho)) * (1.0 + 2e-4)
    assert np.isfinite(Q).all()
    for graph in (True, False):
        S.set_graph(graph)
        S.set_state(Q)
        with pytest.raises(L.LxwError, match=f"element {cell},") as e:
            S.step()
        assert e.value.name == "LXW_ERR_NONFINITE"
    S.set_state(I.random_modal_state(mesh.N, mesh.dim, L.n_modes(mesh.kind, degree), seed=2, amp=0.1))
    S.step()
