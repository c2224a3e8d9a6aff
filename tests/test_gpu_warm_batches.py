"""The warm start's field kernels on batches: a problem's projection and initial
state are the same, bit for bit, whatever number of problems is beside it."""
import numpy as np
import pytest

import warm_reference as R
from lbcases import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a gfx950 GPU")]


@pytest.fixture(scope="module")
def torch():
    import torch
    return torch


@pytest.fixture(scope="module")
def C():
    from paper_1806_10247_amd import capi
    return capi


@pytest.mark.parametrize("L,k2", [(160, 0), (258, 0), (770, 0), (192, 8), (258, 8), (770, 8)])
@pytest.mark.parametrize("planes", [4, 60, 131, 256])
def test_split_projection_by_fewer_workgroups_than_parts(torch, C, L, k2, planes):
    """Up to 256 planes, about 512 workgroups: from all parts of a plane at once to
    two workgroups stepping through them."""
    if planes > 131 and L > 512:
        planes = 140
    g = np.random.default_rng(L + planes)
    a = g.standard_normal((planes, L * L)) + 3.0
    d = torch.from_numpy(a).cuda()
    work = torch.full((C.lb_warm_project_work(planes, L, k2),), float("nan"), dtype=torch.float64, device="cuda")
    C.lb_warm_project_split(d.data_ptr(), planes, L, k2, work.data_ptr())
    assert not torch.isnan(work).any()   # every sum is there
    pick = [0, planes // 2, planes - 1]
    assert np.abs(d[pick].cpu().numpy() - R.remove_staggered(a[pick], L, k2)).max() < 1e-12
    for p in pick:
        one = torch.from_numpy(a[p].copy()).cuda()
        C.lb_warm_project_split(one.data_ptr(), 1, L, k2, work.data_ptr())
        assert torch.equal(one, d[p]), p


@pytest.mark.parametrize("n,B", [(7743, 3), (7744, 3), (9000, 70), (7744, 65537)])
def test_initial_state_of_a_problem_in_a_batch(torch, C, n, B):
    t = torch.Generator(device="cuda").manual_seed(n + B)
    rnd = lambda *s: torch.randn(*s, generator=t, dtype=torch.float64, device="cuda")
    drho, u = rnd(B, n).mul_(1e-3), rnd(2, B, n)   # the velocity serves as the force too: less memory
    rho_out, u_out = torch.empty_like(drho), torch.empty_like(u)
    C.lb_warm_initial_state(drho.data_ptr(), u.data_ptr(), None, u.data_ptr(), None, B, n, 1.0, 1, rho_out.data_ptr(),
                            u_out.data_ptr(), None)
    for b in (0, 1, B // 2, B - 1):
        ub = u[:, b].contiguous()
        r1, u1 = torch.empty(n, dtype=torch.float64, device="cuda"), torch.empty_like(ub)
        C.lb_warm_initial_state(drho[b].data_ptr(), ub.data_ptr(), None, ub.data_ptr(), None, 1, n, 1.0, 1, r1.data_ptr(),
                                u1.data_ptr(), None)
        assert torch.equal(r1, rho_out[b]) and torch.equal(u1, u_out[:, b]), b
