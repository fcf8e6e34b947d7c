"""The direct Poisson solve (full discrete Fourier basis) against the CG without
any pre-solve: phi within kappa tol, no CG iteration needed at the usual
tolerance, E the central differences of phi; on meshes solved in one workgroup
(odd, even, unequal axes, the smallest) and by one launch per axis (tile
remainders along every axis), for both field discretizations.  Where rounding
keeps the residual above the tolerance the CG finishes from the direct
solution and rebuilds E, also for ensemble members one after another; and a
limit on CG iterations below what the pre-solved CG may need keeps the CG."""
import os

import numpy as np
import pytest

from paper_2602_15130_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = 1e-12


def _disc(nc, tol=TOL, op=0, max_iter=20000):
    return {"nc": nc, "np": 6 * nc[0] * nc[1] * nc[2] + 3, "dt": 5e-4, "navg": 1, "cg_tol": tol,
            "cg_max_iter": max_iter, "poisson_op": op}


def _env(name, value, fn):
    old = os.environ.get(name)
    os.environ[name] = value
    try:
        return fn()
    finally:
        if old is None:
            os.environ.pop(name)
        else:
            os.environ[name] = old


def _field_of(phi, nc):
    p = phi.reshape(nc[::-1])
    return np.stack([-(np.roll(p, -1, 2 - d) - np.roll(p, 1, 2 - d)) / (2.0 / nc[d])
                     for d in range(3)]).reshape(3, -1)


def _kappa(nc):
    return max(12.0 / (4.0 * np.sin(np.pi / n) ** 2) for n in nc) * max(nc) ** 2 / min(nc) ** 2


@pytest.mark.parametrize("op", [0, 1])
@pytest.mark.parametrize("nc", [(3, 3, 3), (5, 7, 9), (8, 8, 8), (16, 17, 18), (20, 20, 20),
                                (24, 24, 24), (33, 5, 40), (31, 64, 22), (64, 64, 65)])
def test_direct_solve_matches_cg(nc, op):
    from paper_2602_15130_amd import pic
    prob = W.cfg_problem(two_way=True, collisions=False)
    g = pic.Sim(prob, _disc(nc, op=op), 5, 0)
    h = _env("PIC_CG_LOWMODES", "0", lambda: pic.Sim(prob, _disc(nc, op=op), 5, 0))
    for _ in range(2):
        st = g.stats()
        assert st["cg_iters"] == 0 and st["cg_relres"] <= TOL
        a, b = g.get(pic.STATE_PHI), h.get(pic.STATE_PHI)
        assert np.abs(a - b).max() <= _kappa(nc) * TOL * np.abs(b).max()
        assert abs(a.mean()) <= 1e-14 * np.abs(a).max()
        E = _field_of(a, nc)
        assert np.abs(g.get(pic.STATE_E) - E).max() <= 1e-13 * np.abs(E).max()
        g.step(1)
        h.step(1)


@pytest.mark.parametrize("nc", [(32, 32, 32), (64, 64, 64), (48, 40, 56)])
def test_cg_finishes_where_rounding_stops_the_direct_solve(nc):
    from paper_2602_15130_amd import pic
    prob = W.cfg_problem(two_way=True, collisions=False)
    tol = 1e-15  # near the rounding of the residual
    g = pic.Sim(prob, _disc(nc, tol=tol), 5, 0)
    h = pic.Sim(prob, _disc(nc), 5, 0)
    assert g.stats()["cg_iters"] > 0 and h.stats()["cg_iters"] == 0
    a, b = g.get(pic.STATE_PHI), h.get(pic.STATE_PHI)
    assert np.abs(a - b).max() <= _kappa(nc) * TOL * np.abs(b).max()
    E = _field_of(a, nc)
    assert np.abs(g.get(pic.STATE_E) - E).max() <= 1e-13 * np.abs(E).max()


@pytest.mark.parametrize("tol", [TOL, 1e-15])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_members_one_after_another_equal_single_simulations(precision, tol):
    from paper_2602_15130_amd import pic
    prob = W.cfg_problem(two_way=True, collisions=False)
    disc = _disc((32, 32, 32), tol=tol)
    ens = _env("PIC_CG_MEMBER_LAUNCHES", "1", lambda: pic.Ensemble(prob, disc, 4, 2, 3, precision))
    assert ens.stats()["cg_members_per_launch"] == 1
    assert (ens.stats()["cg_iters"] > 0) == (tol < TOL)
    ens.step(2)
    for m in range(3):
        with pic.Sim(prob, disc, 4, 2 + m, precision) as s:
            s.step(2)
            for item in (pic.STATE_PHI, pic.STATE_E, pic.STATE_V):
                np.testing.assert_array_equal(ens.get(m, item), s.get(item))
    ens.close()


def test_few_allowed_iterations_keep_the_cg():
    from paper_2602_15130_amd import pic
    prob = W.cfg_problem(two_way=True, collisions=False)
    assert pic.Sim(prob, _disc((16, 16, 16), max_iter=63), 5, 0).stats()["cg_iters"] > 0
    assert pic.Sim(prob, _disc((16, 16, 16), max_iter=64), 5, 0).stats()["cg_iters"] == 0
