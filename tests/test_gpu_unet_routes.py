"""The network's routes by size and by stream state: convolutions on 32 x 8 pixel
tiles beyond 16 channels, and inference recorded into a graph of the caller's."""
import numpy as np
import pytest

from lbcases import gpu_available
from oracle import unet as U
from test_gpu_unet import GpuNet, _exact
from test_gpu_unet_layers import _case

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a gfx950 GPU")]

# levels, channels, batch, seed: at 256^2 the first level has 512 tiles of 32 x 8 from batch 2
# and the second (128^2) from batch 8, the number from which they are taken
WIDE = [(2, (32, 64), 2, 1), (2, (48, 32), 2, 0), (2, (64, 32), 2, 0), (1, (96,), 2, 0), (2, (16, 32), 8, 11), (2, (16, 64), 8, 1)]


@pytest.mark.parametrize("levels,ch,B,seed", WIDE)
def test_wide_tiles_beyond_16_channels(levels, ch, B, seed):
    """Integer networks with exact activations and gradients on the oracle: outputs and
    loss bit for bit.  (32, 64): two output tiles a workgroup, 32 and 96 input channels,
    float32 gradients of 32 channels; (48, 32), (64, 32): three and two, 48, 64, 80 and 96;
    (96,): two passes of three; (16, 32), (16, 64): wide tiles on the second level too,
    whose input gradient goes through the pooling into the first.  Weight gradients are float32 sums
    over up to 524,288 pixels: within 1e-5 of the largest, an indexing mistake is of order
    one."""
    net, p, x, t = _case(levels, ch, 5, 2, 256, 256, B, seed)
    acts, rec = [], []
    y, cache = net.forward(p, x, store=lambda a: acts.append(a) or a)
    loss, gy = U.mse(y, t)
    gp, _ = net.backward(p, cache, gy, record=rec)
    assert all(_exact(a) for a in acts) and all(_exact(r) for r in rec) and (y != 0).any()
    assert all((r != 0).any() for r in rec)
    g = GpuNet(net, 256, 256, B)
    try:
        g.C.lb_unet_set_params(g.h, p)
        assert np.array_equal(g.forward(x), y)
        lg, gg = g.loss_grad(x, t)
        assert lg == loss
        assert np.abs(gg - gp).max() <= 1e-5 * np.abs(gp).max()
    finally:
        g.close()


def test_inference_recorded_into_a_graph():
    """lb_unet_forward on a stream that is being recorded: every replay computes the
    output of what the input array holds then, as the eager call does."""
    import torch

    from paper_1806_10247_amd import capi as C
    net = U.UNet(2, (16, 32), 5, 2)
    p, shape = 0.2 * np.random.default_rng(3).standard_normal(net.num_params), (2, 32, 48, 5)
    side = torch.cuda.Stream()
    cfg = C.lb_unet_config_default(levels=2, channels=(16, 32), in_channels=5, out_channels=2, height=32, width=48,
                                   max_batch=2, stream=side.cuda_stream)
    h = C.lb_unet_create(cfg)
    try:
        C.lb_unet_set_params(h, p)
        gen = torch.Generator(device="cuda").manual_seed(1)
        xd = torch.empty(shape, dtype=torch.float32, device="cuda")
        yd, ye = (torch.empty(shape[:3] + (2,), dtype=torch.float32, device="cuda") for _ in range(2))
        torch.cuda.synchronize()
        C.lb_unet_forward(h, xd.data_ptr(), 2, ye.data_ptr())
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            C.lb_unet_forward(h, xd.data_ptr(), 2, yd.data_ptr())
        for _ in range(3):
            xd.copy_(torch.randn(shape, generator=gen, device="cuda"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            C.lb_unet_forward(h, xd.data_ptr(), 2, ye.data_ptr())
            torch.cuda.synchronize()
            assert torch.equal(yd, ye) and bool((yd != 0).any())
    finally:
        C.lb_unet_destroy(h)
