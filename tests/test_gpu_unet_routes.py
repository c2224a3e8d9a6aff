"""The network's routes by size and by stream state: convolutions on 32 x 8 pixel
tiles beyond 16 channels, inference and training recorded into a graph of the
caller's, and what training alone allocates."""
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


def _he(net, seed=3):
    g = np.random.default_rng(seed)
    parts = []
    for co, ci in net.shapes:
        parts += [g.standard_normal(co * 9 * ci) * np.sqrt(2.0 / (9 * ci)), 0.05 * g.standard_normal(co)]
    return np.concatenate(parts)


def test_training_buffers_are_not_an_inference_networks():
    """The weight gradients' split sums (108 MB at this size) are allocated when training
    first runs: a handle that only infers does not hold them."""
    import torch

    from paper_1806_10247_amd import capi as C
    free = lambda: torch.cuda.mem_get_info()[0]
    ch = (16, 32, 32, 48, 48, 48)
    x, y = torch.zeros(16, 256, 256, 13, device="cuda"), torch.zeros(16, 256, 256, 4, device="cuda")
    cfg = C.lb_unet_config_default(levels=6, channels=ch, in_channels=13, out_channels=4, height=256, width=256,
                                   max_batch=16, stream=torch.cuda.current_stream().cuda_stream)
    C.lb_unet_destroy(C.lb_unet_create(cfg))   # what the runtime itself keeps
    torch.cuda.synchronize()
    h = C.lb_unet_create(cfg)
    try:
        C.lb_unet_forward(h, x.data_ptr(), 16, y.data_ptr())
        torch.cuda.synchronize()
        before = free()
        C.lb_unet_loss_grad(h, x.data_ptr(), y.data_ptr(), 16, want_grad=False)
        torch.cuda.synchronize()
        assert before - free() >= 100e6
        after = free()
        C.lb_unet_loss_grad(h, x.data_ptr(), y.data_ptr(), 16, want_grad=False)
        torch.cuda.synchronize()
        assert free() == after
    finally:
        C.lb_unet_destroy(h)


@pytest.mark.parametrize("warm", [False, True])
def test_training_step_recorded_into_a_graph(warm):
    """Gradient and Adam recorded, as a handle's first training call (nothing is allocated
    then: the general path runs) and after an eager one, against the eager call.  With
    eps = 1 and lr = 1 the first update is -g / (|g| + 1): the gradients, each float32
    sums in its path's order over 12,288 pixels, agree to 1e-5 of the largest."""
    import torch

    from paper_1806_10247_amd import capi as C
    net = U.UNet(3, (16, 32, 32), 5, 2)
    p, shape = np.float32(_he(net)), (2, 64, 96, 5)
    gen = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn(shape, generator=gen, device="cuda")
    t = torch.randn(shape[:3] + (2,), generator=gen, device="cuda")
    torch.cuda.synchronize()
    updates = []
    for record in (False, True):
        side = torch.cuda.Stream()
        cfg = C.lb_unet_config_default(levels=3, channels=(16, 32, 32), in_channels=5, out_channels=2, height=64, width=96,
                                       max_batch=2, stream=side.cuda_stream)
        h = C.lb_unet_create(cfg)
        try:
            def step():
                C._ucheck(h, C.lib().lb_unet_loss_grad(h, x.data_ptr(), t.data_ptr(), 2, None, None))
                C.lb_unet_adam(h, 1.0, eps=1.0)

            if warm:
                C.lb_unet_loss_grad(h, x.data_ptr(), t.data_ptr(), 2)
            C.lb_unet_set_params(h, p)
            if record:
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=side):
                    step()
                graph.replay()
            else:
                step()
            updates.append(C.lb_unet_get_params(h).astype(np.float64) - p)
            if record:   # an eager call afterwards allocates and takes the LDS path
                assert np.isfinite(C.lb_unet_loss_grad(h, x.data_ptr(), t.data_ptr(), 2)[1]).all()
        finally:
            C.lb_unet_destroy(h)
    assert np.abs(updates[0]).max() > 1e-2
    assert np.abs(updates[0] - updates[1]).max() <= 1e-5 * np.abs(updates[0]).max()
