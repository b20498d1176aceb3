"""The tangent in the single precision of the mixed-precision solver against
the FP64 one (which the constitutive test compares with the oracle)."""

import numpy as np
import pytest

from gpu_util import make_rve, to_soa
from synthetic import make_microstructure

pytestmark = pytest.mark.gpu

UNIT = 2.0 ** -24


def _tangents(size, seed):
    micro = make_microstructure(24, 12, seed, 0.1)
    rng = np.random.default_rng(seed)
    F = np.eye(3) + size * rng.standard_normal((24 ** 3, 3, 3))
    K = []
    for precision in ("fp64", "mixed"):
        r = make_rve(micro, precision=precision)
        try:
            out = r.debug_constitutive(to_soa(F), 0.1)
        finally:
            r.close()
        assert out["fails"] == 0
        K.append(out["K"])
    return K[0], K[1], micro.law[micro.phase.reshape(-1)] == 1


@pytest.mark.parametrize("size", [1e-4, 1e-3, 5e-3])
def test_particle_tangent_rounding(size):
    """A particle is deformed by its strain alone: an entry of K is one of D,
    rounded once, plus products with H = F - 1 and S2, small against it, and
    two rounded sums: three roundoffs of the largest entry."""
    K, K32, particle = _tangents(size, 5)
    err = np.abs(K32 - K)[:, particle].max(axis=0)
    assert np.max(err / np.abs(K[:, particle]).max(axis=0)) <= 3 * UNIT


def test_elastic_crystal_tangent_rounding():
    """Grains that do not flow: the stored numbers are FP64 ones rounded once
    or sums of a few of those, and so is K : p: two roundoffs in the mean."""
    K, K32, particle = _tangents(1e-4, 6)
    p = np.random.default_rng(7).standard_normal((9, K.shape[1]))
    grain = ~particle

    def apply(A):
        return np.einsum("ijv,jv->iv", A.reshape(9, 9, -1), p)[:, grain]

    err = np.linalg.norm(apply(K32 - K)) / np.linalg.norm(apply(K))
    assert err <= 2 * UNIT
