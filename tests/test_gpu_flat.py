"""The flat step of 3D lattices (casclb_step_flat, chosen for ragged rows and
16-bit storage) against the row kernels (an explicit block_x asks for them):
the same bits, and residuals equal to rounding (their sums run in another
order)."""
import numpy as np
import pytest

import oracle as O
from casclb_inputs import noise
from lbcases import Case, gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a gfx950 GPU")]

SHAPES = [(1, 1, 1), (2, 2, 2), (3, 5, 7), (4, 1, 3), (6, 9, 5), (63, 3, 4), (66, 5, 3), (130, 7, 2), (3, 45, 45)]
WALLS = [(False, False, False), (False, True, True), (True, False, True), (True, True, True)]
REST = {"D3Q27": [np.prod([2 / 3 if d == 0 else 1 / 6 for d in (a % 3, a // 3 % 3, a // 9)]) for a in range(27)],
        "D3Q15": [2 / 9] + [1 / 9] * 6 + [1 / 72] * 8}


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("lattice", ["D3Q27", "D3Q15"])
@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_flat_step_equals_row_step(lattice, i, storage):
    shape = SHAPES[i]
    n = int(np.prod(shape))
    for j, walls in enumerate(WALLS):
        seed = 4 * i + j
        case = Case(lattice, shape, walls=walls, nu=0.06, omega_bulk=1.1, omega_third=0.9, omega_fourth=1.2,
                    force=(2e-5, -1e-5, 1e-5), force_field=noise((3, n), 1e-4, seed=seed) if j % 2 else None,
                    force_time=(O.TIME_COS, 0.02) if j == 2 else (0, 0.0), seed=seed)
        g = np.random.default_rng(seed)
        f = np.array(REST[lattice])[:, None] + 1e-3 * g.standard_normal((len(REST[lattice]), n))
        with case.gpu(storage, residual_interval=4) as flat, case.gpu(storage, residual_interval=4, block_x=64) as row:
            for s in (flat, row):
                s.write_populations(f)
                s.step(13)
            a, b = flat.populations()[0], row.populations()[0]
            assert np.isfinite(a).all()
            assert np.array_equal(a, b), (case, storage, np.abs(a - b).max())
            (ra, na, ta), (rb, nb, tb) = flat.residual(), row.residual()
            assert na == nb and abs(ra - rb) <= 1e-10 * abs(rb)
            # sums of n terms of size <= 1 in two orders of float64
            assert np.allclose(ta, tb, rtol=0, atol=1e-15 * n * len(REST[lattice]))
