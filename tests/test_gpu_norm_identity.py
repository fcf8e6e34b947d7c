"""The error norms compare a particle with the manufactured state of its own
identity: velocities that were moved to another particle together with
everything else the state carries for them (the velocity shape) show in the
velocity norm, in both precision forms and families."""
import numpy as np
import pytest

from paper_2602_15130_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

HEADER = 64  # bytes of a checkpoint before its arrays


@pytest.mark.parametrize("family", ["cfg", "paper"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_velocity_and_shape_of_another_identity_show(precision, family):
    from paper_2602_15130_amd import pic as P
    if family == "cfg":
        prob, disc = W.cfg_problem(two_way=True), W.cfg_disc(8, 4096, 1e-3, 1, 2)
    else:
        prob = W.paper_problem(collisions=True)
        disc = dict(W.paper_level(1), np=4096, navg=2)
    n, dt = disc["np"], np.float64 if precision == "fp64" else np.float32
    with P.Sim(prob, disc, 4, 0, precision) as s:
        before = s.errors()
        raw = bytearray(s.checkpoint())
        # positions (or offsets), velocities, velocity shapes: [3][n] each
        size = 3 * n * np.dtype(dt).itemsize
        v, a = (np.frombuffer(raw, dt, 3 * n, HEADER + k * size).reshape(3, n) for k in (1, 2))
        i, j = int(np.argmax(v[0])), int(np.argmin(v[0]))
        jump = float(v[0, i]) - float(v[0, j])
        for f in (v, a):
            f[:, [i, j]] = f[:, [j, i]]
        s.restore(bytes(raw))
        after = s.errors()
    scale = prob["vbar"]
    eps = np.finfo(dt).eps
    assert before["linf"][3] <= 64 * eps * scale and jump > scale
    np.testing.assert_array_equal(after["linf"][:3], before["linf"][:3])
    assert abs(after["linf"][3] - jump) <= 64 * eps * scale
