"""The direct Poisson solve in three launches (planes, columns) and, where a plane
or an axis does not fit LDS, one launch per transform: the same solution as the
CG within kappa tol, at the edges of the tiles, of the axes' padding to four
and of what fits."""
import numpy as np
import pytest

from test_gpu_direct_solve import TOL, _disc, _env, _field_of, _kappa
from paper_2602_15130_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nc", [(32, 32, 32), (33, 34, 35), (64, 64, 17), (67, 67, 3), (72, 72, 5),
                                (3, 90, 30), (90, 3, 31), (17, 16, 128), (5, 6, 150)])
def test_planes_and_axes_match_cg(nc, precision):
    from paper_2602_15130_amd import pic
    prob = W.cfg_problem(two_way=True, collisions=False)
    with pic.Sim(prob, _disc(nc), 3, 1, precision) as g:
        h = _env("PIC_CG_LOWMODES", "0", lambda: pic.Sim(prob, _disc(nc), 3, 1, precision))
        assert g.stats()["cg_iters"] == 0 and g.stats()["cg_relres"] <= TOL
        a, b = np.asarray(g.get(pic.STATE_PHI)), np.asarray(h.get(pic.STATE_PHI))
        assert np.abs(a - b).max() <= _kappa(nc) * TOL * np.abs(b).max()
        E = _field_of(a, nc)
        assert np.abs(np.asarray(g.get(pic.STATE_E)) - E).max() <= 1e-13 * np.abs(E).max()
        h.close()
