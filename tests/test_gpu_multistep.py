"""Several steps per launch of the 2D lattices (casclb_multistep) against one
step per launch (an explicit block_x asks for the one-step kernels): the same
bits, for lattices that one tile holds whole, that are cut along one axis or
both, with remainders, walls, slices, forcing of every kind and run lengths
from 2 steps to more than one launch."""
import numpy as np
import pytest

import oracle as O
from casclb_inputs import noise
from lbcases import Case, gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a gfx950 GPU")]

# whole in one tile, cut along y, along x, along both; sizes around the tiles' and odd ones
SHAPES = [(4, 64, 1), (1, 1, 1), (2, 3, 5), (32, 32, 1), (31, 33, 2), (5, 300, 1), (300, 5, 1), (61, 67, 1),
          (129, 96, 3), (257, 255, 1), (40, 1000, 1)]
WALLS = [(False, False, False), (False, True, False), (True, False, False), (True, True, False)]
RUNS = [2, 3, 5, 17, 40]


def _case(lattice, shape, walls, seed):
    n = int(np.prod(shape))
    fields = seed % 2 == 0
    return Case(lattice, shape, walls=walls, nu=0.06, D=0.04, omega_bulk=1.1, omega_third=0.9, omega_fourth=1.2,
                omega_phi_high=1.1, force=(2e-5, -1e-5, 0.0), source=2e-5,
                force_field=noise((2, n), 1e-4, seed=seed) if fields else None,
                source_field=noise(n, 1e-4, seed=seed + 1) if fields else None,
                force_time=(O.TIME_COS, 0.02) if seed % 3 == 0 else (0, 0.0),
                source_time=(O.TIME_COS, 0.03) if seed % 4 == 0 else (0, 0.0), seed=seed)


def _state(case):
    g = np.random.default_rng(case.seed + 7)
    w = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)[:, None]
    f = w + 2e-3 * g.standard_normal((9, case.N))
    return f, (0.2 + 2e-2 * g.standard_normal((5, case.N)) if case.lattice == "D2Q9_D2Q5" else None)


def _both(case, storage, setup=lambda s: None, runs=RUNS, **extra):
    f, g = _state(case)
    with case.gpu(storage, residual_interval=23, **extra) as many, \
            case.gpu(storage, residual_interval=23, block_x=64, **extra) as one:
        for s in (many, one):
            setup(s)
            s.write_populations(f, g)
        for n in runs:
            many.step(n)
            one.step(n)
            for a, b in zip(many.populations(), one.populations()):
                if a is not None:
                    assert np.isfinite(a).all()
                    assert np.array_equal(a, b), (case, storage, n, np.abs(a - b).max())
        assert many.residual()[1] == one.residual()[1]


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("lattice", ["D2Q9", "D2Q9_D2Q5"])
@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_several_steps_per_launch_equal_single_steps(lattice, i, storage):
    shape = SHAPES[i]
    for j, walls in enumerate(WALLS):
        _both(_case(lattice, shape, walls, 10 * i + j), storage, runs=RUNS if shape[0] * shape[1] < 20000 else [7, 24])


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("shape", [(3, 64, 1), (70, 66, 1)])
def test_walls_heating_and_lorentz(shape, storage):
    def setup(s):
        s.set_wall_velocity(1, 1, 0.03)
        s.set_scalar_wall(1, 0, 0.0)
        s.set_scalar_wall(1, 1, 1.0)
        s.set_viscous_heating(0.4)
        s.set_lorentz(1e-3)
    _both(_case("D2Q9_D2Q5", shape, (False, True, False), 5), storage, setup)


def test_fields_set_and_cleared_between_runs():
    case = _case("D2Q9_D2Q5", (70, 50, 1), (False, False, False), 2)
    f, g = _state(case)
    with case.gpu("f32") as many, case.gpu("f32", block_x=64) as one:
        for s in (many, one):
            s.write_populations(f, g)
            s.step(9)
            s.set_force_field(None)
            s.step(9)
            s.set_source_field(None)
            s.set_force(1e-5, 0.0)
            s.step(9)
        assert all(np.array_equal(a, b) for a, b in zip(many.populations(), one.populations()))


def test_float16_rounded_to_nearest():
    case = _case("D2Q9_D2Q5", (70, 50, 1), (False, False, False), 2)
    from paper_1806_10247_amd import capi as C
    _both(case, "f16", flags=C.LB_FLAG_F16_NEAREST)
