"""The workgroup-per-cell collision kernel at the edges of its cases: outcomes
of few pairs (many to a wave), around 64 (one to a wave, then several chunks),
up to 192 (earlier pairs in LDS, fewer waves), beyond (earlier pairs in the
cell's scratch, shared by one or several workgroups) and cells whose
accumulators exceed its LDS.  Pair lists equal the serial kernel's; <dv>
differs by the rounding of N_avg FP64 additions (the fixed-point sums are
exact to a quantum far below): 1e-13 of the largest velocity."""
import os

import numpy as np
import pytest

from paper_2602_15130_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _sim(prob, disc, heavy):
    from paper_2602_15130_amd import pic
    old = os.environ.get("PIC_HEAVY")
    os.environ["PIC_HEAVY"] = heavy
    try:
        return pic.Sim(prob, disc, 3, 1)
    finally:
        if old is None:
            os.environ.pop("PIC_HEAVY")
        else:
            os.environ["PIC_HEAVY"] = old


# mean particles per cell, expected pairs per outcome, outcomes
CASES = {"few": (30, 0.5, 5), "one_per_wave": (200, 60.0, 9), "two_waves": (150, 100.0, 6),
         "one_wave": (170, 150.0, 6), "scratch": (700, 260.0, 3), "scratch_whole": (700, 260.0, 64),
         "dense_cells": (3000, 5.0, 300), "pairs_above_n": (90, 230.0, 4)}


@pytest.mark.parametrize("case", list(CASES))
def test_heavy_kernel_equals_serial_kernel(case):
    from paper_2602_15130_amd import pic
    nbar, pairs, navg = CASES[case]
    nc = (3, 4, 3)
    dt = 1e-3
    prob = W.cfg_problem(two_way=True, collisionality=pairs / (0.5 * (nbar - 1) * W.NU_MAX_T / W.T_CFG * dt))
    disc = {"nc": nc, "np": nbar * 36 + 5, "dt": dt, "navg": navg, "cg_tol": 1e-13, "cg_max_iter": 5000}
    g, h = _sim(prob, disc, "1"), _sim(prob, disc, "0")
    cap = int(2.5 * 36 * navg * (pairs + 2))
    for call in (0, 1):
        dg, sg, lg, ng = g.collide(call, 0.0, pairlog_cap=cap)
        dh, sh, lh, nh = h.collide(call, 0.0, pairlog_cap=cap)
        assert ng == nh and 0 < ng <= cap
        lg, lh = (np.asarray(a).reshape(-1, 7) for a in (lg, lh))
        np.testing.assert_array_equal(*(a[np.lexsort((a[:, 3], a[:, 2], a[:, 0]))] for a in (lg, lh)))
        assert np.abs(dg - dh).max() <= 1e-13 * np.abs(g.get(pic.STATE_V)).max()
        # the instance without logs, on the same draws
        p, q = (torch.zeros(3 * disc["np"], dtype=torch.float64, device="cuda") for _ in range(2))
        pic.pic_collide(g.ctx, call, 0.0, p.data_ptr(), q.data_ptr())
        np.testing.assert_array_equal(p.view(3, -1).cpu().numpy(), dg)
    assert g.stats()["n_accepted"] == 2 * h.stats()["n_accepted"]
