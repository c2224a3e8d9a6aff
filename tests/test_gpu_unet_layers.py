"""The LDS convolutions (csrc/nn_conv.hip) at the channel counts and sizes where
they can go wrong: every padded input width above 96, odd raw and output
channel counts, widths that are multiples of 16 but not of 32, one tile, both
tile shapes, and arrays that are not 16-byte aligned.  Integer networks whose
activations (and, where marked, gradients) are exact in bfloat16 on the oracle:
the results must agree bit for bit."""
import numpy as np
import pytest

from lbcases import gpu_available
from oracle import unet as U
from test_gpu_unet import GpuNet, _exact

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a gfx950 GPU")]

# levels, channels, inputs, outputs, H, W, batch, seed, gradients exact
CASES = [(2, (64, 64), 16, 4, 16, 16, 2, 1, True), (2, (96, 96), 9, 16, 16, 32, 2, 52, True),
         (1, (16,), 3, 1, 8, 16, 1, 0, True), (3, (16, 16, 16), 5, 4, 32, 64, 1, 153, True),
         (2, (48, 64), 13, 2, 16, 32, 2, 3, True), (2, (64, 96), 1, 4, 32, 16, 1, 1, True),
         (2, (32, 48), 7, 2, 16, 64, 1, 2, True), (2, (48, 64), 13, 3, 16, 48, 2, 0, False), (2, (64, 96), 1, 5, 32, 16, 1, 0, False),
         (2, (32, 48), 7, 2, 24, 48, 1, 0, False), (1, (16,), 13, 6, 128, 256, 4, 0, False),
         (2, (16, 32), 2, 7, 64, 96, 8, 0, False)]


def _case(levels, ch, cin, cout, H, W, B, seed):
    net = U.UNet(levels, ch, cin, cout)
    g = np.random.default_rng(seed)
    parts = []
    for co, ci in net.shapes:
        pnz = min(0.5, 1.3 / (9 * ci))
        parts.append(g.choice([-1.0, 0.0, 1.0], size=co * 9 * ci, p=[pnz, 1 - 2 * pnz, pnz]))
        parts.append(g.choice([-1.0, 0.0, 1.0], size=co, p=[0.2, 0.5, 0.3]))
    x = g.integers(-2, 3, size=(B, H, W, cin)).astype(np.float64)
    t = g.integers(-4, 5, size=(B, H, W, cout)).astype(np.float64)
    return net, np.concatenate(parts), x, t


@pytest.mark.parametrize("i", range(len(CASES)))
def test_integer_layers_are_bit_exact(i):
    levels, ch, cin, cout, H, W, B, seed, grads = CASES[i]
    net, p, x, t = _case(levels, ch, cin, cout, H, W, B, seed)
    acts, rec = [], []
    y, cache = net.forward(p, x, store=lambda a: acts.append(a) or a)
    assert all(_exact(a) for a in acts) and (y != 0).any()
    g = GpuNet(net, H, W, B)
    try:
        g.C.lb_unet_set_params(g.h, p)
        assert np.array_equal(g.forward(x), y)
        # arrays one float off a 16-byte boundary
        xo = g.torch.empty(x.size + 1, dtype=g.torch.float32, device="cuda")
        yo = g.torch.empty(y.size + 1, dtype=g.torch.float32, device="cuda")
        xo[1:] = g.dev(x).reshape(-1)
        g.C.lb_unet_forward(g.h, xo.data_ptr() + 4, B, yo.data_ptr() + 4)
        assert np.array_equal(yo[1:].cpu().numpy().reshape(y.shape).astype(np.float64), y)
        if grads:
            loss, gy = U.mse(y, t)
            gp, _ = net.backward(p, cache, gy, record=rec)
            assert all(_exact(r) for r in rec)
            lg, gg = g.loss_grad(x, t)
            assert lg == loss and np.array_equal(gg, gp)
    finally:
        g.close()
