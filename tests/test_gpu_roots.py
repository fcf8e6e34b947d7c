"""The inverse distributions of the initial state: every particle's uniforms put
back through the closed form of its CDF (scipy's normal and error functions).
Bounds: the residual of a root is what rounding leaves, a few eps on terms of
order one from the device's CDF, from the root itself and from the host's CDF
(16 eps together); for the normal, relative to the tail probability, eps (1 +
a^2) for each of them."""
import numpy as np
import pytest

from paper_2602_15130_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
special = pytest.importorskip("scipy.special")

EPS = 2.0**-52
NP = 20011


def _state(prob):
    from paper_2602_15130_amd import pic as P
    disc = {"nc": (6, 5, 7), "np": NP, "dt": 1e-3, "navg": 1, "cg_tol": 1e-12, "cg_max_iter": 1000}
    with P.Sim(prob, disc, 3, 1, "fp64") as g:
        pid = np.asarray(g.get(P.STATE_ID))
        return pid, np.asarray(g.get(P.STATE_X)).reshape(3, NP), np.asarray(g.get(P.STATE_V)).reshape(3, NP)


@pytest.mark.parametrize("family", ["cfg", "paper"])
def test_initial_state_solves_its_cdfs(family):
    import oracle as O
    prob = W.cfg_problem() if family == "cfg" else W.paper_problem()
    pid, x, v = _state(prob)
    xi = np.array([O.init_uniforms(3, 1, int(i)) for i in pid]).T
    s = x / np.array(prob["L"])[:, None]
    a = v / np.asarray(O.vhat(prob, 0.0)).reshape(-1, 3)[0][:, None]
    w = 2 * np.pi
    if family == "cfg":
        amp = prob["rho_amp"] * np.sin(w * xi[0]) * np.sin(w * xi[1])
        F = [s[0], s[1], s[2] + amp * (1 - np.cos(w * s[2])) / w]
    else:
        F = [s[0] + 0.2 * (1 - np.cos(w * s[0])) / w,
             s[1] + 0.2 * (np.cos(w * 0.15) - np.cos(w * (s[1] - 0.15))) / w,
             s[2] - (np.cos(w / 15) - np.cos(w * (s[2] + 1 / 15))) / (6 * w)]
    for d in range(3):
        np.testing.assert_allclose(F[d], xi[d], rtol=0, atol=16 * EPS)
        p = np.minimum(xi[3 + d], 1 - xi[3 + d])
        m = -np.abs(a[d])
        assert np.array_equal(a[d] < 0, xi[3 + d] < 0.5)
        if family == "cfg":
            assert np.all(np.abs(special.ndtr(m) - p) <= 16 * EPS * (1 + m * m) * p)
        else:
            G = 0.5 * special.erfc(-m) - m * np.exp(-m * m) / np.sqrt(np.pi)
            np.testing.assert_allclose(G, p, rtol=0, atol=16 * EPS)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nc,np_", [((3, 3, 3), 1), ((3, 4, 5), 300), ((3, 3, 3), 19001),
                                    ((3, 3, 3), 70001), ((16, 16, 16), 4097), ((24, 24, 24), 1500),
                                    ((128, 128, 129), 50001), ((204, 204, 204), 50001)])
def test_initial_state_is_bucketed_and_ordered(nc, np_, precision):
    """Cells of every size (empty, one tile, larger than a tile's LDS slots): the
    particles of a cell in the order of their ids, each in its own cell, and
    velocities that depend on the id alone (bit for bit those of another mesh)."""
    from paper_2602_15130_amd import pic as P

    def state(nc):
        disc = {"nc": nc, "np": np_, "dt": 1e-3, "navg": 1, "cg_tol": 1e-12, "cg_max_iter": 1000}
        with P.Sim(W.cfg_problem(collisions=False), disc, 7, 2, precision) as g:
            return (np.asarray(g.get(P.STATE_ID)), np.asarray(g.get(P.STATE_X)).reshape(3, np_),
                    np.asarray(g.get(P.STATE_V)).reshape(3, np_), np.asarray(g.get(P.STATE_CELL_START)))

    i, x, v, start = state(nc)
    i2, x2, v2, _ = state((4, 3, 5))
    assert np.array_equal(np.sort(i), np.arange(np_)) and start[0] == 0 and start[-1] == np_
    cell = np.repeat(np.arange(len(start) - 1), np.diff(start))
    c = [np.minimum(np.floor(x[d] * nc[d]), nc[d] - 1).astype(int) for d in range(3)]
    assert np.array_equal((c[2] * nc[1] + c[1]) * nc[0] + c[0], cell)
    same = cell[1:] == cell[:-1]
    assert np.all(i[1:][same] > i[:-1][same])
    np.testing.assert_array_equal(v[:, np.argsort(i)], v2[:, np.argsort(i2)])
    if precision == "fp64":
        np.testing.assert_array_equal(x[:, np.argsort(i)], x2[:, np.argsort(i2)])
