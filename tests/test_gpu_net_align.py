"""The network's outputs and targets in arrays that are aligned as floats only
(rows of a larger tensor): the same bits as aligned ones."""

import numpy as np
import pytest

from test_gpu_net import _exact_net, _net, bf16_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [1, 2, 3])
def test_float_aligned_outputs_and_targets(offset):
    import torch
    n = 16
    N = n ** 3
    p, _, X = _exact_net(5, n)
    Xd = torch.from_numpy(bf16_bits(X).view(np.int16).copy()).cuda()
    T = np.zeros((N, 16), dtype=np.float32)
    T[:, :9] = np.random.default_rng(offset).standard_normal((N, 9))

    def shifted(a):
        buf = torch.zeros(N * 16 + offset, device="cuda")
        buf[offset:] = torch.from_numpy(a).cuda().ravel()
        return buf[offset:].view(N, 16)

    net = _net(p)
    try:
        out = shifted(np.zeros((N, 16), dtype=np.float32))
        assert torch.equal(net.forward(Xd, n, out=out), net.forward(Xd, n))
        aligned = torch.from_numpy(T).cuda()
        want = net.train_step(Xd, aligned, n, 0.0, want_grad=True)
        got = net.train_step(Xd, shifted(T), n, 0.0, want_grad=True)
        assert got[0] == want[0] and np.array_equal(got[1], want[1])
        assert net.loss(Xd, shifted(T), n) == want[0]
    finally:
        net.close()
