"""The two elements of an edge form its fluxes each by itself: the same bits up to the sign, on every element
kind, so that what leaves one element enters the other to the last bit."""
import numpy as np
import pytest

import oracle as O
from paper_1601_08145_amd import inputs as I
from paper_1601_08145_amd import lxw as L

pytestmark = pytest.mark.gpu


def case(kind):
    """(library mesh, oracle mesh, degree) with every boundary periodic or transparent."""
    degree = 3 if kind.endswith("3") else 2
    if kind.startswith("line"):
        return L.Mesh.line(300, 0.0, 1.0, 0, 0), O.Mesh.line(300, 0.0, 1.0, 0, 0, degree=degree), degree
    if kind == "quad":
        a = (19, 23, 0.0, 1.0, 0.0, 1.7, [0, 0, 1, 1])
        return L.Mesh.cart(*a), O.Mesh.cart(*a), degree
    if kind == "tet":
        xyz, tet = I.lattice_tets(5, 2)
        return L.Mesh.tet(xyz, tet), O.Mesh.tet(xyz, tet), degree
    xy, tri = I.lattice_delaunay(15, 4)
    return L.Mesh.tri(xy, tri), O.Mesh.tri(xy, tri, degree=degree), degree


@pytest.mark.parametrize("precision", [L.FP64, L.FP32_MIXED])
@pytest.mark.parametrize("kind", ["line", "line3", "quad", "tri", "tri3", "tet"])
def test_both_sides_agree(kind, precision):
    mesh, om, degree = case(kind)
    ei, ki, ej, kj, _ = om.edges()
    inner = ej >= 0
    assert inner.sum() > 200
    S = L.Solver(mesh, degree=degree, precision=precision)
    S.set_debug(True)
    S.set_state(I.random_modal_state(mesh.N, mesh.dim, om.ML, seed=3, amp=0.3, rough_frac=0.3, p_range=(1e-3, 1.0)))
    S.step()
    for stage in (L.STAGE_FLXW, L.STAGE_FLXF):
        f = S.stage(stage)
        a, b = f[ei[inner], ki[inner]], f[ej[inner], kj[inner]]
        assert np.abs(a).max() > 0.0
        print(f"[gpu] {kind} precision {precision} stage {stage}: {(a != -b).sum()} of {a.size} differ", flush=True)
        assert np.array_equal(a, -b)
