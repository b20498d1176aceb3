"""Warm-start network kernels over the grid edges at which their blocks
differ: one tile per wave (16^3, 32^3) and four (48^3 on), blocks that begin
inside a z line (48, 80), one and several voxel groups per weight-gradient
block (from 48^3 on), and an input that is not 16-byte aligned.

The network's arithmetic is exact in bf16 and FP32 (inputs in {-2..2}, about
eight weights of +-1 per output), so forward outputs equal the oracle's bit
for bit.  A gradient is within the bf16 rounding of the back-propagated
signal, (5 - k) 2^-7 times the sum of |x| |dY| over its terms, at layer k.
"""

import numpy as np
import pytest

from oracle import conv
from test_gpu_net import _exact_net, _net, bf16_bits

pytestmark = pytest.mark.gpu


def _device(X, offset=0):
    import torch
    bits = torch.from_numpy(bf16_bits(X).view(np.int16).copy()).cuda()
    if not offset:
        return bits
    buf = torch.zeros(bits.numel() + offset, dtype=torch.int16, device="cuda")
    buf[offset:] = bits.ravel()
    return buf[offset:].view(bits.shape)


def _forward(ps, h):
    for k, (W, b) in enumerate(ps):
        z = conv.conv3d(h, W, b)
        h = np.maximum(z, 0.0) if k < 3 else z
    return h


@pytest.mark.parametrize("n,offset", [(16, 1), (32, 0), (32, 4), (48, 0), (80, 0)])
def test_forward_is_exact(n, offset):
    p, ps, X = _exact_net(21 + n, n)
    ref = _forward(ps, X[:, :40].T.reshape(40, n, n, n).astype(np.float64))
    net = _net(p)
    Y = net.forward(_device(X, offset), n).cpu().numpy()
    net.close()
    assert np.max(np.abs(ref)) > 4.0
    assert np.array_equal(Y[:, :9].astype(np.float64), ref.reshape(9, -1).T)
    assert np.all(Y[:, 9:] == 0.0)


@pytest.mark.parametrize("n,offset", [(32, 1), (48, 0)])
def test_gradients_within_rounding(n, offset):
    import torch
    p, ps, X = _exact_net(33 + n, n)
    rng = np.random.default_rng(n)
    T = np.zeros((n ** 3, 16), dtype=np.float32)
    T[:, :9] = rng.integers(-8, 9, size=(n ** 3, 9))
    net = _net(p)
    Tt, Xt = torch.from_numpy(T).cuda(), _device(X, offset)
    loss, g = net.train_step(Xt, Tt, n, lr=0.0, want_grad=True)
    again, g2 = net.train_step(Xt, Tt, n, lr=0.0, want_grad=True)
    assert np.array_equal(net.get_params(), p)
    net.close()
    assert again == loss and np.array_equal(g, g2)   # sums in a fixed order
    from paper_1806_10599_amd.warmstart import unflatten
    gu = unflatten(g)
    Y, (acts, zs) = conv.Net(ps).forward(
        X[:, :40].T.reshape(40, n, n, n).astype(np.float64))
    diff = Y - T[:, :9].T.reshape(9, n, n, n)
    assert abs(loss - np.mean(diff * diff)) <= 1e-6 * loss
    gz = 2.0 * diff / diff.size
    G = np.abs(gz)
    for k in range(3, -1, -1):
        if k < 3:
            gz, G = gz * (zs[k] > 0), G * (zs[k] > 0)
        W = ps[k][0]
        dX, dW, db = conv.conv3d_backward(acts[k], W, gz)
        dXa, dWa, dba = conv.conv3d_backward(np.abs(acts[k]), np.abs(W), G)
        for got, want, mag in ((gu[k][0], dW, dWa), (gu[k][1], db, dba)):
            assert np.max(np.abs(want)) > 0, k
            assert np.all(np.abs(got - want) <= (5 - k) * 2.0 ** -7 * mag + 1e-12), k
        gz, G = dX, dXa
