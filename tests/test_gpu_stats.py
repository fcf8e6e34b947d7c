"""pic_stats takes its counts and the solver's record in one copy: an ensemble's
are the sums over its members and member 0's record, for one, a few and more
members than the combining workgroup has threads."""
import pytest

from paper_2602_15130_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("members", [1, 3, 260])
def test_stats_of_an_ensemble(members):
    from paper_2602_15130_amd import pic as P
    prob = W.cfg_problem(two_way=True, collisionality=20.0)
    prob["g_max"] = 3.0  # (some pairs are faster)
    disc = {"nc": (4, 4, 4), "np": 700, "dt": 1e-3, "navg": 4, "cg_tol": 1e-12, "cg_max_iter": 15}
    singles = []
    for m in range(min(members, 3)):
        with P.Sim(prob, disc, 5, m, "fp64") as s:
            s.step(2)
            singles.append(s.stats())
    with P.Ensemble(prob, disc, 5, 0, members, "fp64") as e:
        e.step(2)
        st = e.stats()
        again = e.stats()
    assert st == again and st["step"] == 2
    assert st["cg_iters"] == singles[0]["cg_iters"] > 0  # (15 iterations: no direct solve)
    assert st["cg_relres"] == singles[0]["cg_relres"] > 0
    for k in ("n_accepted", "n_gmax"):
        assert singles[0][k] > 0
        if members <= 3:
            assert st[k] == sum(s[k] for s in singles)
        else:
            assert st[k] > 50 * singles[0][k]
