"""The scan of the cell counts with the block sums added up by every workgroup
(one simulation) and scanned in between (an ensemble with more blocks over all
its members than the line): the members equal the simulations bit for bit."""
import numpy as np
import pytest

from paper_2602_15130_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("members", [16, 17])  # 977 blocks each; the line is 16,384
def test_scan_of_an_ensemble_on_a_large_mesh(members):
    from paper_2602_15130_amd import pic as P
    prob = W.cfg_problem(two_way=False, collisions=False)
    disc = {"nc": (100, 100, 100), "np": 70001, "dt": 1e-3, "navg": 1, "cg_tol": 1e-12,
            "cg_max_iter": 5000}
    items = (P.STATE_CELL_START, P.STATE_ID, P.STATE_X, P.STATE_RHO)
    with P.Ensemble(prob, disc, 5, 0, members, "mixed") as e:
        e.step(1)
        for m in (0, members - 1):
            with P.Sim(prob, disc, 5, m, "mixed") as s:
                s.step(1)
                for item in items:
                    np.testing.assert_array_equal(e.get(m, item), s.get(item))
