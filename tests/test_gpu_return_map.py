"""Return mapping over the branches of its residual: integer and non-integer
flow exponents (the smallest integer, the workloads' and a large one), trial
stresses from elastic to a thousand times the critical one, both signs of every
system, the voxel counts at the edges of a wavefront's sixteen voxels and of
the launch rule; and the consistent tangent it feeds."""

import numpy as np
import pytest

from gpu_util import to_soa
from oracle import crystal, material
from synthetic import make_microstructure, material_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [16, 40])   # both sides of the launch rule
@pytest.mark.parametrize("n_exp", [1.0, 3.0, 12.5, 20.0, 37.0])
def test_return_map_matches_oracle(n, n_exp):
    """P and the slips against the oracle's point law.  Both sides stop after
    a Newton step below 1e-10 of the largest slip, which leaves them some
    1e-13 from the root; the stress tolerance is that of the constitutive
    test (1e-12 of max |P|), the slips' 1e-9 of the largest slip."""
    from paper_1806_10599_amd.binding import Rve
    micro = make_microstructure(n, 9, 40 + n, 0.03 if n > 16 else 0.0)
    params = material_params(n_exp=n_exp)
    rng = np.random.default_rng(int(10 * n_exp) + n)
    N = n ** 3
    size = 10.0 ** rng.uniform(-6, -2.2, N)       # strain magnitudes
    H = rng.standard_normal((N, 3, 3)) * size[:, None, None]
    H -= np.trace(H, axis1=1, axis2=2)[:, None, None] / 3 * np.eye(3)
    F = np.eye(3) + H
    r = Rve(n, precision="fp64")
    try:
        r.set_microstructure(micro.phase, micro.quat, micro.law, params)
        got = r.debug_constitutive(to_soa(F), 0.1, tangent=False)
    finally:
        r.close()
    assert got["fails"] == 0
    S0, C = crystal.grain_tables(micro.quat, params)
    cp = np.nonzero(micro.law[micro.phase] == 0)[0][::1 if n == 16 else 11]
    g = micro.phase[cp]
    I = np.broadcast_to(np.eye(3), (cp.size, 3, 3))
    z = np.zeros((cp.size, 12))
    ref = material.cp_update(F[cp], I, z, z, S0[g], C[g], params, 0.1,
                             tangent=False)
    assert ref["ok"].all()
    P = got["P"][:, cp].T.reshape(-1, 3, 3)
    assert np.max(np.abs(P - ref["P"])) <= 1e-12 * np.max(np.abs(ref["P"]))
    dg = got["dg"][:, cp].T
    assert np.max(np.abs(dg - ref["dg"])) <= 1e-9 * np.max(np.abs(ref["dg"]))
