"""The network's routes: inference recorded into a graph of the caller's."""
import numpy as np
import pytest

from lbcases import gpu_available
from oracle import unet as U

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a gfx950 GPU")]

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
