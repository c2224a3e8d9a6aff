"""Batches of small domains (their kernel has no sweeps and no loads ahead)
against the same domains beside a large one (the kernel of every batch): the
same populations, residual steps and stopping, in LDS, partly in LDS and out of
it, at workgroups' edges."""
import numpy as np
import pytest

from lbcases import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a gfx950 GPU")]

SIZES = [(1, 1), (1, 4), (3, 5), (8, 8), (7, 9), (64, 1), (8, 16), (127, 1), (4, 64), (16, 16)]   # up to 256 nodes


def _run(storage, sizes, start, steps, interval, **cfg):
    from paper_1806_10247_amd import capi as C
    domains = [(nx, ny, 0.05 + 0.01 * i, 1e-5, 1e-3 * i) for i, (nx, ny) in enumerate(sizes)]
    b = C.lb_batch_create(C.lb_batch_config_default(storage={"f64": C.LB_STORE_F64, "f32": C.LB_STORE_F32_DEV}[storage],
                                                    check_interval=interval, **cfg), domains)
    try:
        C.lb_batch_init(b)
        for i, f in enumerate(start):
            C.lb_batch_write_populations(b, i, f)
        C.lb_batch_run(b, steps, 0.0)
        done = C.lb_batch_results(b, len(domains))
        out = [np.empty_like(f) for f in start]
        for i, f in enumerate(out):
            C.lb_batch_read_populations(b, i, f)
        return out, done
    finally:
        C.lb_batch_destroy(b)


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("cfg", [dict(block=256), dict(block=256, lds_bytes=8000), dict(block=256, lds_policy=1),
                                 dict(block=64, lds_policy=1), dict(block=1024), dict(block=1024, lds_policy=1)],
                         ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
@pytest.mark.parametrize("steps,interval", [(1, 100), (7, 3), (12, 1)])
def test_small_domains_alone_and_beside_a_large_one(storage, cfg, steps, interval):
    g = np.random.default_rng(steps)
    w = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)[:, None]
    start = [w * (1.0 + 1e-2 * g.standard_normal((9, nx * ny))) for nx, ny in SIZES + [(64, 80)]]
    got, done = _run(storage, SIZES, start[:-1], steps, interval, **cfg)
    want, done1 = _run(storage, SIZES + [(64, 80)], start, steps, interval, **cfg)
    for size, a, b in zip(SIZES, got, want):
        assert np.isfinite(b).all() and np.array_equal(a, b), size
    for a, b in zip(done, done1):   # the same threads add the same nodes in the same order
        assert np.array_equal(a, b[:-1])
