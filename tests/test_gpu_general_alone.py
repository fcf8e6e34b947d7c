"""Loads whose densest cells have more pairs an outcome than a chunk takes: the
general instance alone, chunks first (PIC_LEAN_PASS=0) and the full instance (an
angle log is on) give the same state bit for bit, in steps, captured steps and
collision calls, on both sides of the rule and at a chunk's most pairs."""
import numpy as np
import pytest

from paper_2602_15130_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# mesh, particles per cell, pairs per outcome, outcomes
CASES = {"chunks": ((6, 6, 6), 32, 12.0, 16), "alone": ((6, 6, 6), 32, 30.0, 16),
         "edge_96": ((5, 5, 5), 120, 95.0, 2), "over_96": ((5, 5, 5), 120, 99.0, 3)}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("case", list(CASES))
def test_general_instance_alone(case, precision, monkeypatch):
    from paper_2602_15130_amd import pic as P
    nc, nbar, pairs, navg = CASES[case]
    dt = 1e-4
    prob = W.cfg_problem(two_way=True,
                         collisionality=pairs / (0.5 * (nbar - 0.9) * W.NU_MAX_T / W.T_CFG * dt))
    disc = {"nc": nc, "np": nbar * nc[0] * nc[1] * nc[2] + 3, "dt": dt, "navg": navg, "cg_tol": 1e-12,
            "cg_max_iter": 5000}
    monkeypatch.setenv("PIC_HEAVY", "0")

    def run(env, log=False, graphs=False):
        monkeypatch.delenv("PIC_LEAN_PASS", raising=False)
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        with P.Sim(prob, disc, 4, 1, precision) as s:
            call = s.collide(0, 0.0, pairlog_cap=4 if log else 0)[:2]
            if log:
                s.angle_log(1)
            s.use_graphs(graphs)
            s.step(4)
            return [*call, s.get(P.STATE_X), s.get(P.STATE_V), s.get(P.STATE_ID),
                    np.array(s.stats()["n_accepted"])]

    ref = run({}, log=True)
    assert ref[-1] > 0
    for out in (run({}), run({}, graphs=True), run({"PIC_LEAN_PASS": "0"})):
        for a, b in zip(out, ref):
            np.testing.assert_array_equal(a, b)
