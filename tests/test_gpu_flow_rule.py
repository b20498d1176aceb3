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


def _stress(F, dg, S0, C, Fpi0=None):
    """P at the slips dg in extended precision: in FP64 the elastic strain, a
    difference of numbers of size one, leaves the oracle's P some 5e-16 C11
    from the root, which a soft grain's stress is not large against."""
    F, dg, S0, C = (a.astype(np.longdouble) for a in (F, dg, S0, C))
    A = np.eye(3) - np.einsum("ma,maij->mij", dg, S0)
    if Fpi0 is not None:
        A = np.einsum("mij,mjk->mik", Fpi0.astype(np.longdouble), A)
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


def _compare(n, params, chi_max, hi, seed, every):
    """P, slips and K of a field with plastic strains of 1e-3 and back stresses
    up to chi_max against the oracle on every `every`-th grain voxel: slips to
    1e-9 of the largest, K to 1e-10 of its largest entry.  An FP64 elastic
    strain is a sum of products of numbers of size one: F Fp^-1 three roundings
    of 2^-53 per entry, Fe^T Fe two more, so each strain component is uncertain
    by 5 2^-53 and a stress by that times C11 + 2 |C12|."""
    from paper_1806_10599_amd.binding import Rve
    N = n ** 3
    micro = make_microstructure(n, 9, seed, 0.05 if n > 16 else 0.0)
    rng = np.random.default_rng(seed)
    F = _gradients(rng, N, -6.0, hi)
    Fpi0 = _gradients(rng, N, -5.0, -3.0)
    chi0 = chi_max * np.tanh(rng.standard_normal((N, 12)))
    grain = micro.law[micro.phase.reshape(-1)] == 0
    Fpi0[~grain], chi0[~grain] = np.eye(3), 0.0
    F = np.einsum("mij,mjk->mik", F, np.linalg.inv(Fpi0))  # elastic part: F
    vox = np.nonzero(grain)[0][::every]
    ref = _oracle(micro, vox, F[vox], params, Fpi0[vox], chi0[vox], True)
    assert ref["ok"].all() and np.max(np.abs(ref["dg"])) > 1e-6
    S0, C = crystal.grain_tables(micro.quat, params)
    g = micro.phase.reshape(-1)[vox]
    ref["P"] = _stress(F[vox], ref["dg"], S0[g], C[g], Fpi0[vox])
    r = Rve(n, precision="fp64")
    try:
        r.set_microstructure(micro.phase, micro.quat, micro.law, params)
        r.debug_set_field("Fpinv", to_soa(Fpi0))
        r.debug_set_field("chi", chi0.T)
        got = r.debug_constitutive(to_soa(F), DT)
    finally:
        r.close()
    assert got["fails"] == 0
    rounding = 5 * 2.0 ** -53 * (params[0] + 2 * abs(params[1]))
    for key, rel, floor in (("P", 1e-12, rounding), ("dg", 1e-9, 0.0),
                            ("K", 1e-10, 0.0)):
        want = ref[key].reshape(vox.size, -1)
        err = np.max(np.abs(got[key][:, vox].T - want))
        assert err <= rel * np.max(np.abs(want)) + floor, (key, float(err))


@pytest.mark.parametrize("n", [16, 40])
@pytest.mark.parametrize("kw", [dict(C11=100e3, C12=120e3), dict(C44=-20e3),
                                dict(C44=0.0), dict(C11=121400.0),
                                dict(c_af=-2000.0, d_af=0.0)],
                         ids=["C11<C12", "C44<0", "C44=0", "C11=C12", "softening"])
def test_constants_that_are_not_positive_definite(n, kw):
    """Elastic constants and a back stress that make the local Jacobian
    indefinite or singular moduli vanish are solved like any others."""
    _compare(n, material_params(**kw), 30.0, -3.6, 23, 1 if n == 16 else 13)


@pytest.mark.parametrize("n", [16, 40])
def test_back_stress_beyond_saturation(n):
    """A committed back stress above c/d relaxes: the slips' slopes are
    negative although every constant is positive."""
    _compare(n, material_params(), 150.0, -3.2, 29, 1 if n == 16 else 13)


@pytest.mark.parametrize("n", [16, 32, 40])   # 32^3: the last of a launch rule
@pytest.mark.parametrize("n_exp", [1.0, 3.0, 12.5, 50.0])
def test_state_and_tangent_over_exponents(n, n_exp):
    """P, slips and consistent tangent from a state with plastic strain and
    back stress, for exponents by products and by logarithms; on 32^3 and 40^3
    grains and particles share wavefronts."""
    _compare(n, material_params(n_exp=n_exp), 60.0, -3.2, 31, 1 if n == 16 else 13)
