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
    src, scales = dev(torch, g.standard_normal((4 * B, L * L))), (0.25, 0.5, 1.0)
    fused = torch.empty(4 * B, 4 * L * L, dtype=torch.float64, device="cuda")
    apart = torch.empty_like(fused)
    C.lb_warm_prolong_fields(src.data_ptr(), B, L, scales, fused.data_ptr())
    for p0, planes, s in ((0, B, scales[0]), (B, 2 * B, scales[1]), (3 * B, B, scales[2])):
        C.lb_warm_prolong(src[p0].data_ptr(), planes, L, s, apart[p0].data_ptr())
    assert torch.equal(fused, apart)
    x, y, z = (g.standard_normal((4 * B, L * L)) for _ in range(3))
    a, b, c = ((1.5, 1.25, 0.5), (-0.5, -0.25, 0.75), (0.125, 2.0, -1.0))
    per = lambda w: np.repeat(w, (B, 2 * B, B))[:, None]
    dx, dy, dz, out = (dev(torch, v) for v in (x, y, z, x))
    for third in (False, True):
        C.lb_warm_combine_fields(B, L * L, a, dx.data_ptr(), b, dy.data_ptr(), c if third else None,
                                 dz.data_ptr() if third else None, out.data_ptr())
        terms = [per(a) * x, per(b) * y] + ([per(c) * z] if third else [])
        bound = 3 * EPS * sum(np.abs(t) for t in terms)
        assert (np.abs(out.cpu().numpy() - sum(terms)) <= bound).all()


@pytest.mark.parametrize("L", [64, 66, 128, 130, 258, 1024, 1026, 2048])
@pytest.mark.parametrize("k2", [0, 8])
def test_projection_at_the_edges_of_its_column_groups(torch, C, L, k2):
    a = np.random.default_rng(L).standard_normal((1 if L > 512 else 2, L * L)) + 3.0
    d = dev(torch, a)
    C.lb_warm_project(d.data_ptr(), len(a), L, k2)
    assert np.abs(d.cpu().numpy() - R.remove_staggered(a, L, k2)).max() < 1e-12


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
