"""Warm-start field kernels at the edges of their launch shapes: the fused field
operations against the per-plane ones, the projection where its column groups
change, and the initial state from three launches and in place."""

import numpy as np
import pytest

import warm_reference as R

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.fixture(scope="module")
def C(torch):
    from paper_1806_10247_amd import capi
    return capi


def dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


@pytest.mark.parametrize("L,B", [(2, 1), (17, 3), (128, 1)])
def test_field_operations_match_the_plane_operations(torch, C, L, B):
    g = np.random.default_rng(L)
    y, z = (dev(torch, g.standard_normal((4 * B, L * L))) for _ in range(2))
    x = dev(torch, g.standard_normal((4 * B, 4 * L * L)))
    a, b, c = (1.5, 1.25, 0.5), (-0.5, -0.25, 0.75), (0.125, 2.0, -1.0)
    per = lambda w: dev(torch, np.repeat(w, (B, 2 * B, B))[:, None])
    py, pz, out = (torch.empty_like(x) for _ in range(3))
    C.lb_warm_prolong(y.data_ptr(), 4 * B, L, 1.0, py.data_ptr())
    C.lb_warm_prolong(z.data_ptr(), 4 * B, L, 1.0, pz.data_ptr())
    for first, last in ((False, False), (True, False), (True, True)):
        C.lb_warm_prolong_fields(B, L, a if first else None, x.data_ptr() if first else None, b, y.data_ptr(),
                                 c if last else None, z.data_ptr() if last else None, out.data_ptr())
        terms = [per(b) * py] + ([per(a) * x] if first else []) + ([per(c) * pz] if last else [])
        # a rounding per product and sum of both sides, the prolongations' own are the same or shared
        bound = 4 * EPS * sum(t.abs() for t in terms)
        assert ((out - sum(terms)).abs() <= bound).all()


def test_fields_follow_a_replaced_part(torch, C):
    """Fields of one allocation, one of whose parts is replaced, are what their parts are."""
    from paper_1806_10247_amd import warmstart as W
    g = np.random.default_rng(2)
    L, n = 16, 256
    f = W.Fields(L, 1)
    f.rho.copy_(dev(torch, g.standard_normal(n)))
    f.u = dev(torch, g.standard_normal(2 * n))
    f.phi[:] = 2.0
    whole = W.Fields(L, 1)
    for a, b in ((whole.rho, f.rho), (whole.u, f.u), (whole.phi, f.phi)):
        a.copy_(b)
    fine = W.Fields(2 * L, 1)
    for a, k in ((fine.rho, 1), (fine.u, 2), (fine.phi, 1)):
        a.copy_(dev(torch, g.standard_normal(4 * k * n)))
    apart = W.Fields(2 * L, 1, fine.rho.clone(), fine.u.clone(), fine.phi.clone())
    for x, y in ((W.prolong(f), W.prolong(whole)), (W.extrapolate(fine, f), W.extrapolate(apart, whole)),
                 (W.extrapolate3(fine, whole, W.Fields(L // 2, 1, f.rho[:64], f.u[:128], f.phi[:64]), 0.4, 0.1),
                  W.extrapolate3(apart, whole, W.Fields(L // 2, 1, f.rho[:64], f.u[:128], f.phi[:64]), 0.4, 0.1))):
        for p, q in zip(x.host(), y.host()):
            assert np.abs(p - q).max() <= 8 * EPS * np.abs(q).max()


@pytest.mark.parametrize("L", [64, 66, 128, 130, 258, 1024, 1026, 2048])
@pytest.mark.parametrize("k2", [0, 8])
def test_projection_at_the_edges_of_its_column_groups(torch, C, L, k2):
    a = np.random.default_rng(L).standard_normal((1 if L > 512 else 2, L * L)) + 3.0
    d = dev(torch, a)
    C.lb_warm_project(d.data_ptr(), len(a), L, k2)
    assert np.abs(d.cpu().numpy() - R.remove_staggered(a, L, k2)).max() < 1e-12


@pytest.mark.parametrize("L", [62, 64, 66, 190, 192, 256, 258, 512, 514, 1026, 1538, 2048])
@pytest.mark.parametrize("k2", [0, 1, 8])
def test_split_projection_at_the_edges_of_its_row_parts(torch, C, L, k2):
    a = np.random.default_rng(L).standard_normal((1 if L > 512 else 3, L * L)) + 3.0
    d = dev(torch, a)
    n = C.lb_warm_project_work(len(a), L, k2)
    work = torch.full((n + 64,), float("nan"), dtype=torch.float64, device="cuda")
    if n == 0:   # left to one workgroup per plane
        with pytest.raises(C.LbError):
            C.lb_warm_project_split(d.data_ptr(), len(a), L, k2, work.data_ptr())
        return
    C.lb_warm_project_split(d.data_ptr(), len(a), L, k2, work.data_ptr())
    assert np.abs(d.cpu().numpy() - R.remove_staggered(a, L, k2)).max() < 1e-12
    assert torch.isnan(work[n:]).all()


@pytest.mark.parametrize("n,B", [(4095, 2), (4096, 3), (4161, 2), (65536, 1)])
@pytest.mark.parametrize("inplace", [False, True])
def test_initial_state_in_three_launches_and_in_place(torch, C, n, B, inplace):
    g = np.random.default_rng(n)
    drho, u, phi, F, S = (s * g.standard_normal((k * B, n)) for s, k in ((1e-3, 1), (1e-2, 2), (1.0, 1), (1e-4, 2), (1e-3, 1)))
    r = 1.0 + drho
    un, Fn = u.reshape(2, B, n), F.reshape(2, B, n)
    shift = (r * un).sum(-1) / r.sum(-1)
    want = (r, un - shift[..., None] - Fn / (2 * r), phi - 0.5 * S)
    i = [dev(torch, v) for v in (drho, u, phi, F, S)]
    o = i[:3] if inplace else [torch.empty_like(v) for v in i[:3]]
    C.lb_warm_initial_state(*(v.data_ptr() for v in i), B, n, 1.0, 1, *(v.data_ptr() for v in o))
    # the two sides' sums of n terms each, at worst n roundings of the terms' size, then a few of the node's own
    tol = (4 * EPS, 2 * n * EPS * np.abs(u).max() + 8 * EPS, 8 * EPS * np.abs(phi).max())
    for w, got, t in zip(want, o, tol):
        assert np.abs(got.cpu().numpy().reshape(w.shape) - w).max() <= t
