"""Launch shapes change no bit, on every element kind and in both precisions: the kernels' LDS per lane (up to
138,240 bytes per workgroup of 256 on float32 tetrahedra), their strides and their last workgroups."""
import numpy as np
import pytest

from paper_1601_08145_amd import inputs as I
from paper_1601_08145_amd import lxw as L

pytestmark = pytest.mark.gpu


def case(kind):
    """(mesh, degree): some 600 to 1,000 elements, the last workgroup of every size partly filled."""
    if kind.startswith("line"):
        return L.Mesh.line(777, 0.0, 1.0, 2, 3), 3 if kind == "line3" else 2
    if kind == "quad":
        return L.Mesh.cart(27, 23, 0.0, 1.0, 0.0, 1.0, [3, 1, 2, 2]), 2
    if kind == "tet":
        xyz, tet = I.lattice_tets(6, 0)
        return L.Mesh.tet(xyz, tet, I.boundary_tags_tet(xyz, tet, (0.0, 1.0) * 3, [2, 1, 2, 2, 1, 1])), 2
    xy, tri = I.lattice_delaunay(22, 1)
    return L.Mesh.tri(xy, tri, I.boundary_tags(xy, tri, (0.0, 1.0, 0.0, 1.0), [3, 1, 2, 2])), 3 if kind == "tri3" else 2


@pytest.mark.parametrize("precision", [L.FP64, L.FP32_MIXED])
@pytest.mark.parametrize("kind", ["line", "line3", "quad", "tri", "tri3", "tet"])
def test_shapes_change_no_bit(kind, precision):
    mesh, degree = case(kind)
    Q = I.random_modal_state(mesh.N, mesh.dim, L.n_modes(mesh.kind, degree), 7, rough_frac=0.1, p_range=(1e-3, 1.0))
    out = []
    for shape in (64, 128, 256):
        S = L.Solver(mesh, degree=degree, precision=precision, inflow=(1.0, 0.5, 0.0, 2.5))
        S.set_tune({k: shape for k in ("k_pre", "k_elem", "k_edge", "k_update")})
        S.set_state(Q)
        S.run_steps(6)
        out.append(S.get_state())
    assert np.isfinite(out[0][0]).all()
    for got, t in out[1:]:
        assert np.array_equal(got, out[0][0]) and t == out[0][1]


@pytest.mark.parametrize("precision", [L.FP64, L.FP32_MIXED])
@pytest.mark.parametrize("kind", ["line", "line3", "quad", "tri3", "tet"])
def test_autotune_leaves_the_trajectory(kind, precision):
    mesh, degree = case(kind)
    Q = I.random_modal_state(mesh.N, mesh.dim, L.n_modes(mesh.kind, degree), 8, amp=0.1)
    out = []
    for tuned in (False, True):
        S = L.Solver(mesh, degree=degree, precision=precision, inflow=(1.0, 0.5, 0.0, 2.5))
        S.set_state(Q)
        S.run_steps(2)
        if tuned:
            S.autotune(2)
        S.run_steps(4)
        out.append(S.get_state())
    assert np.array_equal(out[0][0], out[1][0]) and out[0][1] == out[1][1]
