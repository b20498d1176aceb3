"""Point law of the grains where its branches part: powers whose square leaves
the FP64 range, exponents on both routes, states that are not virgin."""

import numpy as np
import pytest

from gpu_util import to_soa
from oracle import crystal, material
from synthetic import make_microstructure, material_params

pytestmark = pytest.mark.gpu

DT = 0.1


def _gradients(rng, N, lo, hi):
    """Isochoric to first order, strain magnitudes 10^lo .. 10^hi."""
    H = rng.standard_normal((N, 3, 3)) * (10.0 ** rng.uniform(lo, hi, N))[:, None, None]
    H -= np.trace(H, axis1=1, axis2=2)[:, None, None] / 3 * np.eye(3)
    return np.eye(3) + H


def _stress(F, dg, S0, C):
    """P at the slips dg of virgin points in extended precision: in FP64 the
    elastic strain, a difference of numbers of size one, leaves the oracle's P
    some 5e-16 C11 from the root, which a soft grain's stress is not large
    against."""
    F, dg, S0, C = (a.astype(np.longdouble) for a in (F, dg, S0, C))
    A = np.eye(3) - np.einsum("ma,maij->mij", dg, S0)
    Fe = np.einsum("mij,mjk->mik", F, A)
    E = (np.einsum("mki,mkj->mij", Fe, Fe) - np.eye(3)) / 2
    S = np.einsum("mijkl,mkl->mij", C, E)
    return np.einsum("mij,mjk,mlk->mil", Fe, S, A)


def _oracle(micro, vox, F, params, Fpi0, chi0, tangent):
    S0, C = crystal.grain_tables(micro.quat, params)
    g = micro.phase.reshape(-1)[vox]
    return material.cp_update(F, Fpi0, chi0, np.zeros((vox.size, 12)), S0[g],
                              C[g], params, DT, tangent=tangent)


@pytest.mark.parametrize("n_exp,g,over", [(50.0, 0.2, 1e3), (64.0, 0.5, 220.0),
                                          (37.0, 0.01, 1.2e4)])
def test_overstress_past_the_range_of_the_power(n_exp, g, over):
    """Trial stresses whose |x|^(2n) is no FP64 number any more, on the points
    that the oracle solves within two thirds of its iteration limit (the
    others, one in fifty, are left undeformed).  Tolerances of the return
    mapping's test: 1e-12 of max |P|, 1e-9 of the largest slip."""
    from paper_1806_10599_amd.binding import Rve
    n = 16
    N = n ** 3
    micro = make_microstructure(n, 9, 17)
    params = material_params(n_exp=n_exp, g=g)
    F = _gradients(np.random.default_rng(int(n_exp)), N, -6.0, -2.5)
    I, z = np.broadcast_to(np.eye(3), (N, 3, 3)), np.zeros((N, 12))
    S0, C = crystal.grain_tables(micro.quat, params)
    ph = micro.phase.reshape(-1)
    ref = _oracle(micro, np.arange(N), F, params, I, z, False)
    easy = ref["ok"] & (ref["iters"] <= 40)
    F = np.where(easy[:, None, None], F, np.eye(3))
    ref["dg"][~easy] = 0.0
    trial = material._cp_eval(F, I, z, z, S0[ph], C[ph], params, DT)["x"]
    assert np.mean(np.max(np.abs(trial), axis=1) > over) > 0.02
    assert easy.mean() > 0.95
    r = Rve(n, precision="fp64")
    try:
        r.set_microstructure(micro.phase, micro.quat, micro.law, params)
        got = r.debug_constitutive(to_soa(F), DT, tangent=False)
    finally:
        r.close()
    assert got["fails"] == 0
    P, dg = got["P"].T.reshape(-1, 3, 3), got["dg"].T
    want = _stress(F, ref["dg"], S0[ph], C[ph])
    assert np.max(np.abs(P - want)) <= 1e-12 * np.max(np.abs(want))
    assert np.max(np.abs(dg - ref["dg"])) <= 1e-9 * np.max(np.abs(ref["dg"]))
