"""The deposit of the unfused step (a wave per cell, chunks of 64 particles): the
charge of a mesh against FP64 sums on the host, for cells with none, few, a
chunk's edge and several chunks of particles.  A node sums fewer than np weights
of at most 1: np eps relative to the largest."""
import numpy as np
import pytest

from paper_2602_15130_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("per_cell", [0, 1, 63, 64, 65, 128, 700])
def test_cells_of_every_size(per_cell, monkeypatch):
    from paper_2602_15130_amd import pic as P
    nc, rng = (4, 3, 5), np.random.default_rng(per_cell)
    np_ = 2 * per_cell + 301
    # two cells with per_cell particles, the others share 301
    c = np.concatenate([np.tile([[1, 2, 3]], (per_cell, 1)), np.tile([[3, 0, 4]], (per_cell, 1)),
                        np.stack([rng.integers(0, n, 301) for n in nc], 1)])
    x = ((c + rng.random((np_, 3))) / nc).T.copy()
    prob = W.cfg_problem(two_way=True, collisions=False)
    disc = {"nc": nc, "np": np_, "dt": 1e-3, "navg": 1, "cg_tol": 1e-12, "cg_max_iter": 1000}
    out = {}
    for unfused in ("1", "0"):
        monkeypatch.setenv("PIC_UNFUSED", unfused)
        with P.Sim(prob, disc, 1, 0, "fp64") as g:
            g.set(P.STATE_X, x)
            out[unfused] = np.asarray(g.get(P.STATE_RHO))
    s = x * np.array(nc)[:, None]
    i = np.floor(s).astype(int)
    o = s - i
    rho = np.zeros(nc[::-1])
    for corner in range(8):
        e = [corner >> d & 1 for d in range(3)]
        w = np.prod([o[d] if e[d] else 1 - o[d] for d in range(3)], axis=0)
        np.add.at(rho, tuple((i[d] + e[d]) % nc[d] for d in (2, 1, 0)), w)
    rho *= prob["q"] * prob["nphys"] / np_ * np.prod(nc)  # charge of a particle over the cell volume
    for r in out.values():
        assert np.abs(r - rho.ravel()).max() <= 4 * np_ * 2.0**-52 * np.abs(rho).max()
