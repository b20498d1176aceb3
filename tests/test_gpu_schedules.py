"""Which FFT schedules exist, and that the one with the largest tiles runs on
each edge: its blocks hold the most LDS (107 KB on 128^3 in single precision
and on 64^3 in double)."""

import pytest

from synthetic import make_microstructure, material_params, macro_F

pytestmark = pytest.mark.gpu

EDGES = [16, 24, 32, 40, 48, 64, 96, 128]
# largest edge with three components per slab block, with sixteen kz columns
CPB3 = {"fp64": 48, "mixed": 64}
TT16 = {"fp64": 64, "mixed": 128}
EINVAL = -1


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", EDGES)
def test_the_schedules_of_an_edge(n, precision):
    from paper_1806_10599_amd.binding import Rve, RveError
    r = Rve(n, precision=precision)
    try:
        for cpb in (1, 2, 3):
            for tt in (4, 8, 12, 16):
                exists = (cpb != 2 and tt != 12
                          and (cpb == 1 or n <= CPB3[precision])
                          and (tt < 16 or n <= TT16[precision]))
                if exists:
                    r.set_fft_schedule(cpb, tt)
                    continue
                with pytest.raises(RveError) as e:
                    r.set_fft_schedule(cpb, tt)
                assert e.value.code == EINVAL
    finally:
        r.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", EDGES)
def test_the_largest_schedule_runs(n, precision):
    """The same Newton and CG counts (one per solve apart at most) as with the
    smallest tiles, K:p folded in and not."""
    from paper_1806_10599_amd.binding import Rve
    micro = make_microstructure(n, 6, 70 + n)
    sched = (3 if n <= CPB3[precision] else 1, 16 if n <= TT16[precision] else 8)
    ref = None
    for s in ((1, 4, 0), sched + (0,), sched + (1,)):
        r = Rve(n, precision=precision, newton_tol=1e-5)
        try:
            r.set_microstructure(micro.phase, micro.quat, micro.law,
                                 material_params())
            r.set_fft_schedule(*s)
            info = r.increment(macro_F(0.001), 0.1)
        finally:
            r.close()
        assert info["status"] == 0 and info["cg_iters_total"] > 0
        ref = ref or info
        assert info["newton_iters"] == ref["newton_iters"]
        for a, b in zip(info["cg_iters"], ref["cg_iters"]):
            assert abs(a - b) <= 1


@pytest.mark.parametrize("use_graph", [False, True])
def test_batches_with_different_tiles_side_by_side(use_graph):
    """What one batch's blocks take of the LDS does not limit another's: a
    batch with 107 KB goes on after one with 81 KB was set up."""
    from paper_1806_10599_amd.binding import BatchRve
    first, second = (BatchRve([n], precision="fp64", use_graph=use_graph)
                     for n in (64, 48))
    try:
        for b, n in ((first, 64), (second, 48)):
            micro = make_microstructure(n, 6, n)
            b.set_microstructure(0, micro.phase, micro.quat, micro.law,
                                 material_params())
            b.set_fft_schedule(n, 1, 16)
            info, = b.increment(macro_F(0.0005), 0.1)
            assert info["status"] == 0 and info["cg_iters_total"] > 0
        info, = first.increment(macro_F(0.001), 0.1)
        assert info["status"] == 0 and info["cg_iters_total"] > 0
    finally:
        first.close()
        second.close()
