"""What a query of an ensemble checks is put together over all members on the
device: the flag of a solve that cannot converge reaches every query, for one,
a few and more members than the combining workgroup has threads; and queries of
members without a flag return their states."""
import numpy as np
import pytest

from paper_2602_15130_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("members", [1, 2, 17, 300])
@pytest.mark.parametrize("converges", [True, False])
def test_flags_of_all_members_reach_a_query(members, converges):
    from paper_2602_15130_amd import pic as P
    prob = W.cfg_problem(two_way=True, collisions=False)
    disc = {"nc": (4, 4, 4), "np": 256, "dt": 1e-3, "navg": 1, "cg_tol": 1e-12,
            "cg_max_iter": 20000 if converges else 1}
    with P.Ensemble(prob, disc, 5, 0, members, "fp64") as e:
        e.step(2)
        if converges:
            for m in (0, members - 1):
                with P.Sim(prob, disc, 5, m, "fp64") as s:
                    s.step(2)
                    np.testing.assert_array_equal(e.get(m, P.STATE_X), s.get(P.STATE_X))
            r = e.errors()
            assert r["status"] == P.PIC_OK and r["l2"].shape == (members, 7)
        else:
            for query in (lambda: e.get(members - 1, P.STATE_RHO), e.errors, e.stats):
                with pytest.raises(P.PicError) as ei:
                    query()
                assert ei.value.code == P.PIC_ENOCONV
