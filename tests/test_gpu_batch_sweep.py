"""Batch domains stepped several at a time through LDS rings, or in place in LDS,
against the same domains stepped one at a time in global memory: bit for bit, at
the edges of the rings, of a workgroup's nodes and of the check interval."""

import numpy as np
import pytest

from lbcases import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a gfx950 GPU")]

# (nx, ny): one and two nodes per thread and one more; wide, narrow and the widest a ring takes with 1024 threads
SIZES = [(20, 20), (32, 32), (25, 41), (32, 64), (3, 683), (1, 2500), (2, 1281), (3, 1025), (64, 70), (40, 128), (250, 41),
         (256, 17), (257, 17), (496, 9), (497, 9)]


def _run(storage, domains, start, block, policy, steps, interval):
    from paper_1806_10247_amd import capi as C
    cfg = C.lb_batch_config_default(storage={"f64": C.LB_STORE_F64, "f32": C.LB_STORE_F32_DEV}[storage],
                                    check_interval=interval, block=block, lds_policy=policy)
    b = C.lb_batch_create(cfg, domains)
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
@pytest.mark.parametrize("block", [64, 1024])
@pytest.mark.parametrize("steps,interval", [(1, 100), (2, 100), (3, 100), (7, 100), (13, 4), (5, 1), (12, 3), (11, 5)])
def test_sweeps_match_single_steps(storage, block, steps, interval):
    g = np.random.default_rng(steps + 100 * interval)
    w = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)[:, None]
    domains = [(nx, ny, 0.05 + 0.01 * i, 1e-5, 1e-3 * i) for i, (nx, ny) in enumerate(SIZES)]
    start = [w * (1.0 + 1e-2 * g.standard_normal((9, nx * ny))) for nx, ny in SIZES]
    got, (st, res, status) = _run(storage, domains, start, block, 0, steps, interval)
    want, (st1, res1, status1) = _run(storage, domains, start, block, 1, steps, interval)
    for size, a, b in zip(SIZES, got, want):
        assert np.isfinite(b).all() and np.array_equal(a, b), size
    assert np.array_equal(st, st1) and np.array_equal(status, status1)
    # the same terms, float64, in another order
    n = max(nx * ny for nx, ny in SIZES)
    assert np.array_equal(np.isinf(res), np.isinf(res1))
    fin = ~np.isinf(res1)
    assert (np.abs(res[fin] - res1[fin]) <= 2 * n * np.finfo(np.float64).eps * np.abs(res1[fin])).all()
