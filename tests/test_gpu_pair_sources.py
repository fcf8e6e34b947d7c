"""Where a pass takes its candidate pairs from changes no bit: lists drawn before
the pass (PIC_LEAN_PASS=1), chunks drawn in the tile (=0), the full instance
(an angle log is on), and in FP64 the separate kernels.  At the edges of each:
tiles of many nearly empty cells, N_avg no multiple of four, several pairs per
outcome, more than a list's four, a list that overflows, several chunks and
several blocks of (cell, outcome) items, outcomes at and over the 64 pairs of a
chunk, cells larger than a tile's LDS slots; passes of both halves and of one."""
import numpy as np
import pytest

from paper_2602_15130_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# mesh, mean particles per cell, expected pairs per outcome, outcomes
CASES = {"sparse": ((9, 8, 7), 2, 0.05, 6), "few": ((8, 8, 8), 32, 0.06, 16),
         "several": ((8, 8, 8), 32, 1.3, 5), "over_four": ((6, 6, 6), 40, 4.2, 3),
         "overflow": ((8, 8, 8), 32, 0.9, 20), "chunks": ((6, 6, 6), 30, 2.0, 70),
         "items": ((8, 8, 8), 6, 0.3, 40), "edge_64": ((5, 5, 5), 120, 63.0, 2),
         "over_64": ((5, 5, 5), 120, 66.0, 2), "large_cells": ((3, 3, 3), 700, 1.0, 3)}


def _setup(case):
    nc, nbar, pairs, navg = CASES[case]
    dt = 1e-3
    prob = W.cfg_problem(two_way=True,
                         collisionality=pairs / (0.5 * (nbar - 0.9) * W.NU_MAX_T / W.T_CFG * dt))
    n = nc[0] * nc[1] * nc[2]
    return prob, {"nc": nc, "np": nbar * n + 3, "dt": dt, "navg": navg, "cg_tol": 1e-13,
                  "cg_max_iter": 5000}


def _state(monkeypatch, prob, disc, precision, env, log=False):
    from paper_2602_15130_amd import pic as P
    monkeypatch.setenv("PIC_HEAVY", "0")
    for k in ("PIC_LEAN_PASS", "PIC_UNFUSED"):
        monkeypatch.delenv(k, raising=False)
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    with P.Sim(prob, disc, 4, 1, precision) as s:
        if log:
            s.angle_log(1)
        for n in (1, 3):
            s.step(n)
        out = [s.get(i) for i in (P.STATE_X, P.STATE_V, P.STATE_ID, P.STATE_PHI)]
        st = s.stats()
        return out + [np.array([st["n_accepted"], st["n_gmax"]])]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("case", list(CASES))
def test_pair_sources_agree(case, precision, monkeypatch):
    prob, disc = _setup(case)
    ref = _state(monkeypatch, prob, disc, precision, {}, log=True)
    assert ref[-1][0] > 0
    others = [{"PIC_LEAN_PASS": "1"}, {"PIC_LEAN_PASS": "0"}]
    if precision == "fp64":
        others.append({"PIC_UNFUSED": "1"})
    for env in others:
        for a, b in zip(_state(monkeypatch, prob, disc, precision, env), ref):
            np.testing.assert_array_equal(a, b, err_msg=str(env))


@pytest.mark.parametrize("collisions", [True, False])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("case", ["sparse", "several", "overflow", "chunks", "large_cells"])
def test_collision_calls_agree(case, precision, collisions, monkeypatch):
    """pic_collide without a pair log (drawn lists or chunks) against the one with
    a log (the full instance), also on a problem that steps without collisions."""
    from paper_2602_15130_amd import pic as P
    prob, disc = _setup(case)
    prob["collisions"] = int(collisions)
    monkeypatch.setenv("PIC_HEAVY", "0")
    for lean in ("1", "0"):
        monkeypatch.setenv("PIC_LEAN_PASS", lean)
        with P.Sim(prob, disc, 4, 1, precision) as s:
            for call in (0, 1):
                a = s.collide(call, 0.0)
                b = s.collide(call, 0.0, pairlog_cap=4)
                np.testing.assert_array_equal(a[0], b[0])
                np.testing.assert_array_equal(a[1], b[1])
                assert np.abs(a[0]).max() > 0
