"""The kernel timing hook of a handle that has picked no schedule (none was
needed yet, or the choice was reset) times every pass."""

import numpy as np
import pytest

from gpu_util import make_rve
from synthetic import macro_F, make_microstructure

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_every_kernel_is_timed_without_a_schedule(precision):
    r = make_rve(make_microstructure(16, 6, 3), precision=precision)
    try:
        assert r.increment(macro_F(1e-3), 0.1)["status"] == 0
        r.set_fft_schedule(0, 0)
        ms = r.bench_kernels(2)
        assert all(np.isfinite(v) and v > 0.0 for v in ms.values()), ms
        assert r.increment(macro_F(2e-3), 0.1)["status"] == 0
    finally:
        r.close()
