"""Small meshes run whole steps in one workgroup: the same bits as the separate launches, at the sizes
around its workgroup sizes and its limits, over several kernels' worth of steps, to an end time, and with every
form of the moment limiter and the wave speed."""
import numpy as np
import pytest

from paper_1601_08145_amd import inputs as I
from paper_1601_08145_amd import lxw as L

pytestmark = pytest.mark.gpu


def line(n, degree, precision, bc=(2, 3), **kw):
    mesh = L.Mesh.line(n, 0.0, 1.0, *bc)
    Q = I.random_modal_state(n, 1, L.n_modes(L.LINE, degree), n, amp=0.3, rough_frac=0.2, p_range=(1e-3, 1.0))
    return mesh, Q, dict(degree=degree, precision=precision, cfl=0.05, inflow=(1.0, 0.5, 0.0, 2.5), **kw)


def tri(n, precision, **kw):
    xy, t = I.lattice_delaunay(n, n)
    tags = I.boundary_tags(xy, t, (0.0, 1.0, 0.0, 1.0), [3, 1, 2, 2])
    Q = I.random_modal_state(len(t), 2, 6, n, amp=0.3, rough_frac=0.2, p_range=(1e-3, 1.0))
    return L.Mesh.tri(xy, t, tags), Q, dict(precision=precision, inflow=(1.0, 0.5, 0.0, 2.5), **kw)


def both(mesh, Q, kw, steps, T=None):
    out = []
    for graph in (True, False):
        S = L.Solver(mesh, **kw)
        S.set_state(Q)
        S.set_graph(graph)
        st = None
        if T is None:
            S.run_steps(steps)
            S.sync()
        else:
            st = S.advance(T)
        got, t = S.get_state()
        out.append((got, t, st.steps if st else steps))
    assert np.isfinite(out[0][0]).all()
    assert np.array_equal(out[0][0], out[1][0]) and out[0][1:] == out[1][1:]
    return out[0]


@pytest.mark.parametrize("degree", [2, 3])
@pytest.mark.parametrize("precision", [L.FP64, L.FP32_MIXED])
@pytest.mark.parametrize("n", [2, 63, 256, 257, 511, 512, 513])
def test_line(n, degree, precision):
    both(*line(n, degree, precision), 12)


@pytest.mark.parametrize("precision", [L.FP64, L.FP32_MIXED])
@pytest.mark.parametrize("n", [2, 9, 12, 13])  # 2, 128, 242 and (separate launches) 288 triangles
def test_triangles(n, precision):
    both(*tri(n, precision), 12)


@pytest.mark.parametrize("exact", [0, 1])
@pytest.mark.parametrize("speed", [L.SPEED_POINTS, L.SPEED_AVERAGES])
@pytest.mark.parametrize("shock", [L.SHOCK_OFF, L.SHOCK_PLAIN])
def test_forms(exact, speed, shock):
    kw = dict(theta_exact=exact, wave_speed=speed, shock=shock)
    both(*line(100, 2, L.FP64, **kw), 8)
    both(*tri(9, L.FP64, **kw), 8)


def test_end_time_and_many_steps():
    mesh, Q, kw = line(40, 2, L.FP64, bc=(0, 0))
    got = both(mesh, Q, kw, 0, T=0.05)
    assert got[1] == 0.05 and got[2] > 20
    S = L.Solver(mesh, **kw)
    S.set_state(Q)
    S.run_steps(1500)  # two kernels
    S.sync()
    R = L.Solver(mesh, **kw)
    R.set_state(Q)
    for _ in range(1500):
        R.step()
    assert np.array_equal(S.get_state()[0], R.get_state()[0])


def test_errors_name_the_element():
    """An average that is not positive: reported as by the separate launches, the solver usable after."""
    mesh, Q, kw = line(100, 2, L.FP64, bc=(1, 1))
    for graph in (True, False):
        S = L.Solver(mesh, **kw)
        bad = Q.copy()
        bad[37, 0, 0] = -1.0
        S.set_state(bad, checked=False)
        S.set_graph(graph)
        with pytest.raises(L.LxwError, match="element 37") as e:
            S.step()
        assert e.value.code == -5
        S.set_state(Q)
        S.step()
