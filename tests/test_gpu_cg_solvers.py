"""The CG solvers of a run without the direct solve (a number of low modes is
asked for, PIC_CG_LOWMODES): how many members one launch takes."""
import pytest

from paper_2602_15130_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = 1e-13


def _disc(nc, tol=TOL, op=0, per_cell=4):
    n = nc[0] * nc[1] * nc[2]
    return {"nc": nc, "np": per_cell * n + 3, "dt": 5e-4, "navg": 1, "cg_tol": tol,
            "cg_max_iter": 20000, "poisson_op": op}


def _sim(monkeypatch, prob, disc, env, members=0):
    from paper_2602_15130_amd import pic as P
    for k in ("PIC_CG_LOWMODES", "PIC_CG_GLOBAL", "PIC_CG_BLOCKS", "PIC_CG_INSTANCE",
              "PIC_CG_PLAIN_LAUNCH", "PIC_CG_MEMBER_LAUNCHES"):
        monkeypatch.delenv(k, raising=False)
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    return P.Ensemble(prob, disc, 5, 0, members, "fp64") if members else P.Sim(prob, disc, 5, 0, "fp64")


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
