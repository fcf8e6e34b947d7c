"""Pairs drawn by a workgroup per tile (hundreds of outcomes on a small mesh)
against the full instance, which draws in the tile (an angle log is on): the
same state bit for bit, for single simulations in both forms, ensembles and
captured steps, with N_avg no multiple of four and with lists that overflow."""
import numpy as np
import pytest

from paper_2602_15130_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# mesh, particles per cell, pairs per outcome, outcomes (64 items a tile and call: the line)
CASES = {"line": ((8, 8, 8), 32, 0.05, 32), "below": ((8, 8, 8), 32, 0.05, 28),
         "many": ((8, 8, 8), 32, 0.005, 1023), "thousands": ((4, 5, 6), 32, 0.001, 4096),
         "overflow": ((6, 6, 6), 32, 0.06, 210), "sparse": ((9, 8, 7), 2, 0.01, 90)}


def _run(case, precision, graphs=False, log=False, members=0):
    from paper_2602_15130_amd import pic as P
    nc, nbar, pairs, navg = CASES[case]
    prob = W.cfg_problem(two_way=True,
                         collisionality=pairs / (0.5 * (nbar - 0.9) * W.NU_MAX_T / W.T_CFG * 1e-3))
    disc = {"nc": nc, "np": nbar * nc[0] * nc[1] * nc[2] + 3, "dt": 1e-3, "navg": navg,
            "cg_tol": 1e-12, "cg_max_iter": 5000}
    items = (P.STATE_X, P.STATE_V, P.STATE_ID, P.STATE_PHI)
    if members:
        with P.Ensemble(prob, disc, 4, 0, members, precision) as e:
            e.step(6)
            return [[e.get(m, i) for i in items] for m in range(members)]
    with P.Sim(prob, disc, 4, 0, precision) as s:
        if log:
            s.angle_log(1)
        s.use_graphs(graphs)
        s.step(6)
        return [s.get(i) for i in items] + [np.array(s.stats()["n_accepted"])]


@pytest.fixture(autouse=True)
def lists(monkeypatch):
    monkeypatch.setenv("PIC_HEAVY", "0")
    monkeypatch.setenv("PIC_LEAN_PASS", "1")


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("case", list(CASES))
def test_pairs_drawn_by_tile(case, precision):
    ref = _run(case, precision, log=True)
    assert ref[-1] > 0
    for graphs in (False, True):
        for a, b in zip(_run(case, precision, graphs=graphs), ref):
            np.testing.assert_array_equal(a, b)


def test_pairs_drawn_by_tile_in_ensembles():
    ref = _run("many", "mixed", log=True)
    ens = _run("many", "mixed", members=3)
    for a, b in zip(ens[0], ref):
        np.testing.assert_array_equal(a, b)
    assert not np.array_equal(ens[1][1], ens[0][1])
