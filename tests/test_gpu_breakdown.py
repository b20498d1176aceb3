"""A CG run that ends without a direction: stiffnesses so large that the
single-precision vectors overflow make p . (K : p) infinite or NaN, and the
run breaks down in its first iteration."""

import numpy as np
import pytest

from synthetic import make_microstructure

pytestmark = pytest.mark.gpu

F_BAR = np.eye(3) + 0.02 * np.arange(9.0).reshape(3, 3) / 9


def _statev(n, scale):
    stiff = make_microstructure(n, 6, 3).phase.reshape(-1) % 2 == 1
    k = scale * np.where(stiff, 6.0, 1.0)
    return np.stack([k, 1.5 * k, np.zeros(n ** 3)])


def _rve(n, scale, **kw):
    from paper_1806_10599_amd.binding import Rve
    r = Rve(n, precision="mixed", newton_tol=1e-6, **kw)
    r.set_user_material("neo_hooke", _statev(n, scale))
    return r


@pytest.mark.parametrize("use_graph", [False, True])
def test_iterate_survives_an_infinite_direction(use_graph):
    """The Newton iteration goes on from the finite iterate (here zero): the
    residual stays the predictor's, and no voxel's F becomes NaN."""
    r = _rve(16, 1e36, newton_max_iter=3, use_graph=use_graph)
    try:
        info = r.increment(F_BAR, 1.0)
        assert info["status"] == -4                      # not converged
        assert info["cg_breakdowns"] == info["newton_iters"] == 3
        assert info["local_failures"] == 0
        assert info["residuals"][0] > 1e-3
        assert info["residuals"] == [info["residuals"][0]] * 4
        assert np.all(r.field("F") == np.eye(3).reshape(9, 1))
    finally:
        r.close()


def test_tuning_after_a_breakdown():
    """The vectors that a broken run left do not reach the solve in which the
    schedule is picked again."""
    n = 16
    r, fresh = _rve(n, 1e36, newton_max_iter=2), _rve(n, 8e4)
    try:
        assert r.increment(F_BAR, 1.0)["cg_breakdowns"] == 2
        r.set_user_material("neo_hooke", _statev(n, 8e4))
        r.set_fft_schedule(0, 0)
        got, want = r.increment(F_BAR, 1.0), fresh.increment(F_BAR, 1.0)
        assert want["status"] == 0
        assert got["cg_breakdowns"] == 0
        assert got["cg_iters"][0] == want["cg_iters"][0]
        assert abs(got["residuals"][1] / want["residuals"][1] - 1) < 1e-3
    finally:
        r.close()
        fresh.close()
