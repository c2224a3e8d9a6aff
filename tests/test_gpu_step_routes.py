"""lb_step's routes: steps that a caller records and replays, and settings that
change the route between runs."""
import numpy as np
import pytest

from lbcases import Case, gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a gfx950 GPU")]


def _state(case):
    g = np.random.default_rng(case.seed + 7)
    w = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)[:, None]
    f = w + 2e-3 * g.standard_normal((9, case.N))
    return f, (0.2 + 2e-2 * g.standard_normal((5, case.N)) if case.lattice == "D2Q9_D2Q5" else None)


@pytest.mark.parametrize("steps", [2, 6, 10, 12, 300])
@pytest.mark.parametrize("lattice,shape,storage", [("D2Q9", (4, 64, 1), "f64"), ("D2Q9_D2Q5", (70, 66, 1), "f32"),
                                                   ("D2Q9_D2Q5", (200, 300, 1), "f64"), ("D2Q9", (128, 130, 2), "f32")])
def test_recorded_steps_replayed(lattice, shape, storage, steps):
    """An even number of plain steps recorded once: every replay continues from the
    state that the replay before left, whatever number of launches the steps took
    (eager steps of another context say what it is, bit for bit)."""
    import torch
    case = Case(lattice, shape, walls=(False, True, False), nu=0.06, D=0.04, force=(2e-5, -1e-5, 0.0), source=2e-5, seed=3)
    f, g = _state(case)
    side = torch.cuda.Stream()
    with case.gpu(storage, residual_interval=0, stream=side.cuda_stream) as rec, \
            case.gpu(storage, residual_interval=0, block_x=64) as one:
        for s in (rec, one):
            s.write_populations(f, g)
            s.step(steps)
            s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            rec.step(steps)
        for _ in range(4):
            graph.replay()
            torch.cuda.synchronize()
            one.step(steps)
            for a, b in zip(rec.populations(), one.populations()):   # eager work between the replays
                if a is not None:
                    assert np.array_equal(a, b), np.abs(a - b).max()


@pytest.mark.parametrize("steps", [4, 10, 80])
@pytest.mark.parametrize("lattice,shape,cfg", [("D3Q27", (12, 10, 9), {}), ("D3Q15", (64, 5, 6), {}),
                                               ("D2Q9", (70, 66, 1), {"block_x": 64})])
def test_recorded_single_steps_replayed(lattice, shape, cfg, steps):
    """The same where every step is a launch: runs that would replay a step graph are
    recorded launch by launch."""
    import torch
    case = Case(lattice, shape, nu=0.06, force=(2e-5, -1e-5, 1e-5), seed=3)
    f0 = case.perturbed_state(case.oracle())[0]
    side = torch.cuda.Stream()
    with case.gpu("f64", residual_interval=0, stream=side.cuda_stream, **cfg) as rec, \
            case.gpu("f64", residual_interval=0, **cfg) as one:
        for s in (rec, one):
            s.write_populations(f0)
            s.step(steps)
            s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            rec.step(steps)
        for _ in range(3):
            graph.replay()
            torch.cuda.synchronize()
            one.step(steps)
            assert np.array_equal(rec.populations()[0], one.populations()[0])


@pytest.mark.parametrize("lattice,shape,walls", [("D2Q9_D2Q5", (1024, 1030, 1), (False, True, False)),
                                                 ("D2Q9_D2Q5", (1001, 1000, 1), (True, True, False)),
                                                 ("D2Q9", (96, 11000, 1), (False, True, False))])
def test_float16_steps_as_walls_are_set_and_cleared(lattice, shape, walls):
    """Moving walls make large float16 lattices take one step per launch, and resting
    ones several again: the same bits as single launches throughout."""
    case = Case(lattice, shape, walls=walls, nu=0.06, D=0.04, force=(2e-5, -1e-5, 0.0), source=2e-5, seed=4)
    f, g = _state(case)
    with case.gpu("f16", residual_interval=9) as s, case.gpu("f16", residual_interval=9, block_x=64) as one:
        for c in (s, one):
            c.write_populations(f, g)
        for speed in (0.0, 0.03, 0.0):
            for c in (s, one):
                c.set_wall_velocity(1, 1, speed)
                c.step(11)
            for a, b in zip(s.populations(), one.populations()):
                if a is not None:
                    assert np.array_equal(a, b), np.abs(a - b).max()
            assert s.residual()[1] == one.residual()[1]


def _kernel(lattice, shape, storage, walls=(False, False, False), setup=lambda s: None, **cfg):
    with Case(lattice, shape, walls=walls).gpu(storage, residual_interval=0, **cfg) as s:
        setup(s)
        info = s.info()
        return info.step_kernel.decode(), info.block_x


def test_info_names_the_kernel_of_the_steps():
    """lb_get_info names the kernel that plain steps run, for every kind of route."""
    from paper_1806_10247_amd import capi as C
    for st, tag in (("f64", "f64"), ("f32", "f32dev"), ("f16", "f16dev")):
        for lat in ("D2Q9", "D2Q9_D2Q5"):
            assert _kernel(lat, (64, 64, 1), st)[0] == f"casclb_multistep<{lat},{tag}>"
            assert _kernel(lat, (64, 64, 1), st)[1] in (256, 512, 1024)
            assert _kernel(lat, (63, 64, 1), st, block_x=64) == (f"casclb_step<{lat},{tag}>", 64)
            assert _kernel(lat, (64, 64, 1), st, rows_per_thread=2)[0] == f"casclb_step<{lat},{tag}>"
        for lat in ("D3Q27", "D3Q15"):
            assert _kernel(lat, (63, 20, 20), st) == (f"casclb_step_flat<{lat},{tag}>", 64)
            assert _kernel(lat, (63, 20, 20), st, block_x=128) == (f"casclb_step<{lat},{tag}>", 128)
    assert _kernel("D3Q27", (64, 20, 20), "f64")[0] == "casclb_step<D3Q27,f64>"
    assert _kernel("D3Q27", (128, 20, 20), "f32")[0] == "casclb_step<D3Q27,f32dev>"
    assert _kernel("D3Q27", (64, 20, 20), "f16")[0] == "casclb_step_flat_pair<D3Q27,f16dev>"
    assert _kernel("D3Q15", (64, 20, 20), "f16")[0] == "casclb_step_flat<D3Q15,f16dev>"
    assert _kernel("D3Q27", (64, 20, 20), "f16", x_pairs=2)[0] == "casclb_step_xpair<D3Q27,f16dev>"
    assert _kernel("D2Q9", (64, 64, 1), "f16", x_pairs=2)[0] == "casclb_step_xpair<D2Q9,f16dev>"
    # large float16 lattices with a moving wall take one step per launch, and several again without
    moving, y = (lambda s: s.set_wall_velocity(1, 1, 0.1)), (False, True, False)
    assert _kernel("D2Q9_D2Q5", (2048, 1024, 1), "f16", y)[0] == "casclb_multistep<D2Q9_D2Q5,f16dev>"
    assert _kernel("D2Q9_D2Q5", (2048, 1024, 1), "f16", y, moving)[0] == "casclb_step_xpair<D2Q9_D2Q5,f16dev>"
    assert _kernel("D2Q9_D2Q5", (2048, 1024, 1), "f32", y, moving)[0] == "casclb_multistep<D2Q9_D2Q5,f32dev>"
    assert _kernel("D2Q9_D2Q5", (256, 256, 1), "f16", y, moving)[0] == "casclb_multistep<D2Q9_D2Q5,f16dev>"
    with Case("D2Q9_D2Q5", (2048, 1024, 1), walls=y).gpu("f16", residual_interval=0) as s:
        for speed, kernel in ((0.1, "casclb_step_xpair"), (0.0, "casclb_multistep"), (0.1, "casclb_step_xpair")):
            s.set_wall_velocity(1, 1, speed)
            assert s.info().step_kernel.decode() == f"{kernel}<D2Q9_D2Q5,f16dev>"
    assert _kernel("D2Q9", (64, 64, 1), "f64", flags=C.LB_FLAG_XCD_REMAP)[0] == "casclb_multistep<D2Q9,f64>"


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("lattice,shape,walls", [("D2Q9", (4, 64, 1), (False, True, False)),
                                                 ("D2Q9_D2Q5", (70, 66, 1), (False, False, False)),
                                                 ("D2Q9_D2Q5", (257, 130, 3), (True, True, False))])
def test_poison_covers_the_several_step_launches(lattice, shape, walls, storage):
    """LB_FLAG_DEBUG_POISON on a lattice that takes several steps per launch: the same
    kernel, every node written by it, the padding of the buffer it wrote poisoned."""
    import torch

    from paper_1806_10247_amd import capi as C
    case = Case(lattice, shape, walls=walls, nu=0.06, D=0.04, force=(2e-5, -1e-5, 0.0), source=2e-5, seed=5)
    f, g = _state(case)
    plane = case.N + 24
    need = plane * (14 if g is not None else 9) * {"f64": 8, "f32": 4, "f16": 2}[storage]
    bufs = [torch.zeros(need, dtype=torch.uint8, device="cuda") for _ in range(2)]
    flags = C.LB_FLAG_DEBUG_POISON | C.LB_FLAG_EXTERNAL_BUFFERS
    with case.gpu(storage, residual_interval=7, flags=flags, plane_pad=24) as p, \
            case.gpu(storage, residual_interval=7, plane_pad=24) as s:
        C.lb_bind_buffers(p.ctx, bufs[0].data_ptr(), bufs[1].data_ptr(), need)
        assert p.info().step_kernel == s.info().step_kernel and b"multistep" in p.info().step_kernel
        for c in (p, s):
            c.write_populations(f, g)
            c.step(11)   # six steps, a check, four steps
        for a, b in zip(p.populations(), s.populations()):
            if a is not None:
                assert np.isfinite(a).all() and np.array_equal(a, b)
        (rp, np_, tp), (rs, ns, ts) = p.residual(), s.residual()
        assert rp == rs and np_ == ns and np.array_equal(tp, ts)
        dt = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}[storage]
        now = next(b for b in bufs if b.data_ptr() == p.info().buf_current).view(dt).view(-1, plane)
        assert torch.isfinite(now[:, :case.N]).all() and torch.isnan(now[:, case.N:]).all()


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("lattice,shape,walls,fields", [("D2Q9", (300, 45, 1), (False, True, False), False),
                                                        ("D2Q9_D2Q5", (37, 29, 1), (True, True, False), False),
                                                        ("D2Q9", (64, 48, 1), (False, False, False), True),
                                                        ("D2Q9_D2Q5", (64, 40, 1), (False, False, False), True),
                                                        ("D2Q9_D2Q5", (32, 8, 3), (False, False, False), False)])
def test_step_graphs_single_launches_and_several_steps_agree(lattice, shape, walls, fields, storage):
    """2D lattices over runs of both parities and lengths, with residual checks: an
    explicit block_x and forcing constant in time replays step graphs, a cos(0 t) factor
    launches every step by itself, and the automatic shape takes several steps per launch.
    The same bits."""
    from casclb_inputs import noise
    n = int(np.prod(shape))
    out = []
    for time, cfg, kernel in (((0, 0.0), {"block_x": 64}, b"casclb_step<"), ((1, 0.0), {"block_x": 64}, b"casclb_step<"),
                              ((0, 0.0), {}, b"casclb_multistep<")):
        case = Case(lattice, shape, walls=walls, nu=0.06, D=0.03, omega_bulk=1.1, force=(1e-5, -2e-5, 0.0), source=1e-5,
                    force_field=noise((2, n), 1e-4, seed=1) if fields else None,
                    source_field=noise(n, 1e-4, seed=2) if fields else None, force_time=time, source_time=time, seed=6)
        f, g = _state(case)
        with case.gpu(storage, residual_interval=70, **cfg) as s:
            assert s.info().step_kernel.startswith(kernel)
            s.write_populations(f, g)
            for steps in (333, 97, 29, 140):
                s.step(steps)
            out.append(s.populations() + (s.residual(),))
    for got in out[1:]:
        for a, b in zip(out[0][:2], got[:2]):
            if a is not None:
                assert np.isfinite(a).all() and np.array_equal(a, b)
        (r0, n0, t0), (r1, n1, t1) = out[0][2], got[2]
        # the automatic shape's blocks differ: sums of n terms of size <= 1 in two orders of float64
        assert n0 == n1 and abs(r0 - r1) <= 1e-10 * abs(r0) and np.allclose(t0, t1, rtol=0, atol=1e-15 * n * 14)


def test_flat_and_row_contexts_take_their_routes():
    """The sizes that the flat and the several-step kernels are compared with the rows at
    do run those kernels."""
    import test_gpu_flat as F
    import test_gpu_multistep as M
    for st in ("f64", "f32", "f16"):
        for lat in ("D3Q27", "D3Q15"):
            for shape in F.SHAPES:
                assert _kernel(lat, shape, st)[0].startswith("casclb_step_flat")
                assert _kernel(lat, shape, st, block_x=64)[0].startswith(("casclb_step<", "casclb_step_xpair<"))
        for lat in ("D2Q9", "D2Q9_D2Q5"):
            for shape in M.SHAPES:
                assert _kernel(lat, shape, st)[0].startswith("casclb_multistep<")
                assert _kernel(lat, shape, st, block_x=64)[0].startswith(("casclb_step<", "casclb_step_xpair<"))
