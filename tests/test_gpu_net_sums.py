"""Rounding of the network's gradients over large grids: sums of up to two
million equal terms, which single precision holds exactly for a thousand of
them but not for sixteen thousand."""

import numpy as np
import pytest

from paper_1806_10599_amd.warmstart import param_count, unflatten
from test_gpu_net import _net, bf16_round

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64, 96, 128])
def test_gradient_of_a_constant_field(n):
    """Biases alone feed the layers, so activations (a2, a3) and
    back-propagated signals (b, c) are constant and a gradient is their
    product times the number of voxels.  Products have at most 16 significant
    bits: over 64^3 and 128^3, powers of two, every partial sum of a sound
    accumulation is exact; over 96^3 sums may be rounded twice to single
    precision."""
    import torch
    N = n ** 3
    a2, a3 = 255.0 / 128, 253.0 / 128
    p = np.zeros(param_count(), dtype=np.float32)
    off, views = 0, []
    for ci, co in ((40, 32), (32, 32), (32, 32), (32, 9)):
        W, off = p[off:off + 27 * ci * co].reshape(27, ci, co), off + 27 * ci * co
        views.append((W, p[off:off + co]))
        off += co
    views[1][1][:] = a2
    views[2][1][:] = a3
    views[3][0][13] = 2.0 ** -5          # centre tap: Y = a3 in every channel
    step = 187.0 / 128                   # Y - T
    T = torch.zeros(N, 16, device="cuda")
    T[:, :9] = a3 - step
    X = torch.zeros(N, 48, dtype=torch.int16, device="cuda")
    b = bf16_round(np.float32(2.0 * step / (9.0 * N)))
    c = bf16_round(np.float32(9 * b * 2.0 ** -5))
    net = _net(p)
    try:
        loss, g = net.train_step(X, T, n, lr=0.0, want_grad=True)
    finally:
        net.close()
    gu = unflatten(g)
    assert abs(loss - step ** 2) <= 1e-12 * step ** 2
    tol = 0.0 if n != 96 else 2.0 ** -23
    for layer, want in ((3, N * a3 * b), (2, N * a2 * c)):
        assert np.all(np.abs(gu[layer][0] - want) <= tol * want), layer
    assert np.all(np.abs(gu[2][1] - N * c) <= tol * N * c)
