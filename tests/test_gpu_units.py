"""The solution does not depend on the unit of length: G is invariant to a
common factor of the wave vectors, and a power of two changes no digit."""

import numpy as np
import pytest

from synthetic import make_microstructure, material_params, macro_F

pytestmark = pytest.mark.gpu

L = np.array([1.0, 1.5, 0.7])


def _params():
    """The workloads' constants in Pa."""
    p = np.array(material_params(), dtype=np.float64)
    p[[0, 1, 2, 4, 6, 8]] *= 1e6      # C11, C12, C44, g, c, E
    return p


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("power", [-50, 50])
def test_increment_is_invariant_to_the_unit_of_length(precision, power):
    from paper_1806_10599_amd.binding import BatchRve, Rve
    n = 24
    micro = make_microstructure(n, 6, 11, 0.05)
    out = []
    for scale in (1.0, 2.0 ** power):
        kw = dict(L=tuple(scale * L), projection="continuous",
                  precision=precision)
        r, b = Rve(n, **kw), BatchRve([n], **kw)
        try:
            r.set_fft_schedule(1, 4, 0)          # sums in the same order
            b.set_fft_schedule(n, 1, 4)
            args = micro.phase, micro.quat, micro.law, _params()
            r.set_microstructure(*args)
            b.set_microstructure(0, *args)
            info = r.increment(macro_F(0.002), 0.1)
            binfo, = b.increment(macro_F(0.002), 0.1)
            assert info["status"] == binfo["status"] == 0
            assert info["cg_breakdowns"] == binfo["cg_breakdowns"] == 0
            out.append((info["cg_iters"], binfo["cg_iters"], r.field("F"),
                        r.field("P"), b.field(0, "F")))
        finally:
            r.close()
            b.close()
    for one, other in zip(*out):
        assert np.array_equal(one, other)
