"""The CG solvers and the low-mode pre-solve, run for their own iterations: with a
number of low modes asked for (PIC_CG_LOWMODES) there is no direct solve before
them, and every side that is meant to iterate is seen to.  The on-chip brick
solver against the global-memory one, the pre-solve against none in both field
discretizations, ordinary against cooperative launches, one launch per ensemble
member against one for all; and how many members one launch takes."""
import numpy as np
import pytest

import oracle as O
from paper_2602_15130_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = 1e-13
MODES = "24"  # the default number of low modes per axis


def _disc(nc, tol=TOL, op=0, per_cell=4):
    n = nc[0] * nc[1] * nc[2]
    return {"nc": nc, "np": per_cell * n + 3, "dt": 5e-4, "navg": 1, "cg_tol": tol,
            "cg_max_iter": 20000, "poisson_op": op}


def _kappa(nc):
    return max(12.0 / (4.0 * np.sin(np.pi / n) ** 2) for n in nc) * max(nc) ** 2 / min(nc) ** 2


def _sim(monkeypatch, prob, disc, env, members=0):
    from paper_2602_15130_amd import pic as P
    for k in ("PIC_CG_LOWMODES", "PIC_CG_GLOBAL", "PIC_CG_BLOCKS", "PIC_CG_INSTANCE",
              "PIC_CG_PLAIN_LAUNCH", "PIC_CG_MEMBER_LAUNCHES"):
        monkeypatch.delenv(k, raising=False)
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    return P.Ensemble(prob, disc, 5, 0, members, "fp64") if members else P.Sim(prob, disc, 5, 0, "fp64")


def _close(a, b, nc):
    from paper_2602_15130_amd import pic as P
    pa, pb = a.get(P.STATE_PHI), b.get(P.STATE_PHI)
    assert np.abs(pa - pb).max() < _kappa(nc) * TOL * np.abs(pb).max()


@pytest.mark.parametrize("nc,env", [((16, 16, 16), {}), ((32, 32, 32), {}),
                                    ((32, 32, 32), {"PIC_CG_BLOCKS": "16"}), ((64, 64, 64), {}),
                                    ((64, 64, 64), {"PIC_CG_INSTANCE": "4,1024"}),
                                    ((96, 96, 96), {}), ((128, 128, 128), {}), ((64, 32, 16), {})])
def test_brick_solver_iterates_as_the_global_one(nc, env, monkeypatch):
    prob = W.cfg_problem(two_way=True, collisions=False)
    disc = _disc(nc)
    g = _sim(monkeypatch, prob, disc, dict(env, PIC_CG_LOWMODES="0"))
    h = _sim(monkeypatch, prob, disc, {"PIC_CG_LOWMODES": "0", "PIC_CG_GLOBAL": "1"})
    for _ in range(2):
        sg, sh = g.stats(), h.stats()
        assert sg["cg_brick"][0] > 0 and sh["cg_brick"] == [0, 0, 0]
        assert sg["cg_iters"] > 10 and abs(sg["cg_iters"] - sh["cg_iters"]) <= 1
        assert max(sg["cg_relres"], sh["cg_relres"]) <= TOL
        _close(g, h, nc)
        g.step(1)
        h.step(1)
    if nc == (16, 16, 16):
        o = O.Sim(prob, disc, 5, 0)
        assert o.init() == 0 and o.step(2) == 0
        po = o.get(o.PHI)
        from paper_2602_15130_amd import pic as P
        assert np.abs(g.get(P.STATE_PHI) - po).max() < _kappa(nc) * TOL * np.abs(po).max()


@pytest.mark.parametrize("op", [0, 1])
@pytest.mark.parametrize("nc", [(16, 16, 16), (12, 10, 14), (64, 64, 64), (48, 40, 56)])
def test_low_mode_presolve_saves_iterations(nc, op, monkeypatch):
    prob = W.cfg_problem(two_way=True, collisions=False)
    disc = _disc(nc, op=op)
    # (modes that leave some to the CG on the small meshes too)
    g = _sim(monkeypatch, prob, disc, {"PIC_CG_LOWMODES": MODES if min(nc) > 40 else "3"})
    h = _sim(monkeypatch, prob, disc, {"PIC_CG_LOWMODES": "0"})
    for _ in range(2):
        a, b = g.stats()["cg_iters"], h.stats()["cg_iters"]
        assert 0 < a < b
        _close(g, h, nc)
        g.step(1)
        h.step(1)


@pytest.mark.parametrize("glob", ["0", "1"])
def test_launch_forms_change_no_bit(glob, monkeypatch):
    """Ordinary launches, and one launch per member, where the CG iterates."""
    from paper_2602_15130_amd import pic as P
    prob = W.cfg_problem(two_way=True, collisions=False)
    nc = (32, 32, 32)
    base = {"PIC_CG_LOWMODES": "3", "PIC_CG_GLOBAL": glob}
    disc = _disc(nc)
    ref = _sim(monkeypatch, prob, disc, base)
    plain = _sim(monkeypatch, prob, disc, dict(base, PIC_CG_PLAIN_LAUNCH="1"))
    together = _sim(monkeypatch, prob, disc, base, members=3)
    each = _sim(monkeypatch, prob, disc, dict(base, PIC_CG_MEMBER_LAUNCHES="1"), members=3)
    assert each.stats()["cg_members_per_launch"] == 1 < together.stats()["cg_members_per_launch"]
    for s in (ref, plain, together, each):
        s.step(2)
        assert s.stats()["cg_iters"] > 5
    for item in (P.STATE_PHI, P.STATE_E, P.STATE_X):
        a = ref.get(item)
        np.testing.assert_array_equal(plain.get(item), a)
        np.testing.assert_array_equal(together.get(0, item), a)
        for m in range(3):
            np.testing.assert_array_equal(each.get(m, item), together.get(m, item))


def test_members_of_one_solver_launch(monkeypatch):
    """The plain solver's registers leave room for four workgroups of 256 threads
    with two nodes each a CU: 120 members of eight workgroups each run in one
    launch on 256 CUs."""
    if torch.cuda.get_device_properties(0).multi_processor_count < 256:
        pytest.skip("fewer CUs")
    prob = W.cfg_problem(two_way=True, collisions=False)
    e = _sim(monkeypatch, prob, _disc((16, 16, 16), per_cell=1), {"PIC_CG_LOWMODES": "3"}, members=120)
    st = e.stats()
    assert st["cg_brick"][0] > 0 and st["cg_blocks"] == 8
    assert st["cg_members_per_launch"] == 120
