"""lb_step and HIP graphs: steps that a caller records and replays."""
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
