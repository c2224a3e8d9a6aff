"""Timed workloads of the framework: what its users run, through its public entry points.

Four families, each over the range of sizes it is used at:

  flow     the fused cascaded step (`Solver.step`) of D2Q9, D2Q9 + D2Q5 and D3Q27 lattices, from the
           paper's small channels and ducts to the 256^3 duct, in every storage type, with uniform
           forces, force / source fields and oscillating forcing, periodic and walled, with and
           without the residual read between blocks of steps;
  batch    independent Hartmann channels advanced together (`lb_batch_run`);
  network  the warm-start network: inference and one training step (`Surrogate`, `lb_unet_*`);
  fields   the warm start's field pipeline between the coarse solves and the fine iteration
           (`warmstart`: guess, level differences, network input, estimate, initial state).

`listed` names the fixed cases, `draw` takes another one of the same ranges, `prepare` builds what a
program holds before the call, `run` is one pass, `work` its unavoidable bytes and operations and
`exact` the same outputs from plain float64 torch.
"""
import math

import numpy as np
import torch

from paper_1806_10247_amd import capi as C
from paper_1806_10247_amd import warmstart as W
from paper_1806_10247_amd.solver import Solver

_ELEM = {"f64": 8, "f32": 4, "f16": 2}
_TORCH = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}
_DIMS = {"D2Q9": 2, "D2Q9_D2Q5": 2, "D3Q27": 3}
_Q = {"D2Q9": 9, "D2Q9_D2Q5": 14, "D3Q27": 27}
# operations per node and step: moment sweeps, shifts, relaxation and back
_NODE_FLOPS = {"D2Q9": 250, "D2Q9_D2Q5": 330, "D3Q27": 950}
_ON_CHIP = 256 << 20   # a state of at most this many bytes can stay in the last-level cache between steps


def _flow(name, lattice, shape, storage, steps, walls="", force="uniform", interval=0):
    nx, ny, nz = shape
    return dict(name=name, family="flow", lattice=lattice, nx=nx, ny=ny, nz=nz, storage=storage, steps=steps,
                walls=walls, force=force, interval=interval)


def _network(name, kind, L, batch, levels=6, width=16, features="levels"):
    return dict(name=name, family="network", kind=kind, L=L, batch=batch, levels=levels, width=width,
                features=features)


def listed():
    return [
        # the paper's Poiseuille channel, run to its steady profile in blocks of steps
        _flow("channel_4x64_f64", "D2Q9", (4, 64, 1), "f64", 200, walls="y", interval=100),
        # the paper's square duct (3 x 45 x 45 nodes)
        _flow("duct_3x45x45_f64", "D3Q27", (3, 45, 45), "f64", 100, walls="yz", interval=100),
        # a coarse level of the warm start: one residual interval, then both residuals are read
        _flow("coarse_64_f32", "D2Q9_D2Q5", (64, 64, 1), "f32", 100, force="field", interval=100),
        # the warm start's fine iteration at its own size
        _flow("fine_256_f32", "D2Q9_D2Q5", (256, 256, 1), "f32", 100, force="field", interval=100),
        # flow and scalar on a lattice of no convenient size under an oscillating force
        _flow("coupled_1531x1021_f64", "D2Q9_D2Q5", (1531, 1021, 1), "f64", 20, force="cos"),
        # the benchmark's duct
        _flow("duct_256_f32", "D3Q27", (256, 256, 256), "f32", 10, walls="yz"),
        # a forced periodic box in the compact storage, rows that no block size divides
        _flow("box_250x203x190_f16", "D3Q27", (250, 203, 190), "f16", 10, force="field"),
        # a parameter sweep of Hartmann channels
        dict(name="hartmann_512_f32", family="batch", domains=512, steps=200, storage="f32", interval=100),
        # one problem's correction: the network as a warm start calls it
        _network("network_forward_1", "forward", 256, 1),
        # corrections of a batch of problems
        _network("network_forward_16", "forward", 256, 16),
        # one step of the network's training: loss, gradient, Adam
        _network("network_train_16", "train", 256, 16),
        # one problem's fields between its coarse solves and its fine iteration
        dict(name="warm_fields_256", family="fields", L=256, batch=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["2d", "2d", "2d", "3d", "3d", "batch", "forward", "forward", "train", "fields"])
    if kind == "2d":
        lattice = rng.choice(["D2Q9", "D2Q9_D2Q5", "D2Q9_D2Q5"])
        nx, ny = _log(rng, 3, 1600), _log(rng, 16, 1600)
        nz = rng.choice([1, 1, 1, _log(rng, 2, 16)])
        if nx * ny * nz > 1 << 21:
            nz = 1
        case = _flow("", lattice, (nx, ny, nz), rng.choice(["f64", "f32", "f32", "f16"]),
                     0, walls=rng.choice(["", "", "y", "xy"]), force=rng.choice(["uniform", "field", "cos"]),
                     interval=rng.choice([0, 50, 100]))
        most = 200
    elif kind == "3d":
        nx, ny, nz = _log(rng, 3, 256), _log(rng, 12, 256), _log(rng, 12, 256)
        case = _flow("", "D3Q27", (nx, ny, nz), rng.choice(["f64", "f32", "f32", "f16"]), 0,
                     walls=rng.choice(["", "y", "yz"]), force=rng.choice(["uniform", "field"]),
                     interval=rng.choice([0, 50]))
        most = 100
    elif kind == "batch":
        return dict(family="batch", domains=_log(rng, 32, 512), steps=rng.randint(100, 200),
                    storage=rng.choice(["f32", "f32", "f64"]), interval=50)
    elif kind in ("forward", "train"):
        levels = rng.choice([3, 4, 6])
        side = 4 << (levels - 1)
        case = _network("", kind, side * max(1, _log(rng, 64, 256) // side), _log(rng, 1, 16), levels,
                        rng.choice([16, 16, 32]), rng.choice(["guess", "levels"]))
        del case["name"]
        return case
    else:
        return dict(family="fields", L=rng.choice([64, 96, 128, 160, 256, 320, 512]), batch=_log(rng, 1, 4))
    # about as many node updates as the listed cases of this kind at most
    nodes = case["nx"] * case["ny"] * case["nz"]
    case["steps"] = max(2, min(rng.randint(most // 2, most), int(3e7 if kind == "2d" else 8e7) // nodes))
    del case["name"]
    return case


# ---------------------------------------------------------------------------
# inputs, from the seed alone
# ---------------------------------------------------------------------------

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 13)


def _uniform(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _smooth(g, shape, count, amplitude):
    """`count` fields [count][N], each a sum of four sinusoids of at most `amplitude` (x fastest)."""
    axes = [torch.arange(n, device="cuda", dtype=torch.float64) * (2.0 * math.pi / n) for n in shape]
    out = torch.zeros(count, shape[2], shape[1], shape[0], device="cuda", dtype=torch.float64)
    for c in range(count):
        for _ in range(4):
            k = torch.randint(1, 4, (3,), generator=g, device="cuda").tolist()
            a = _uniform(g, -0.25 * amplitude, 0.25 * amplitude, 4).tolist()
            wave = [torch.sin(k[i] * axes[i] + 25.0 * a[i] / amplitude) for i in range(3)]
            out[c] += a[3] * wave[0] * wave[1][:, None] * (wave[2] if shape[2] > 1 else 1.0 + 0 * wave[2])[:, None, None]
    return out.reshape(count, -1)


def _flow_inputs(case, seed):
    g = _generator(seed)
    shape = (case["nx"], case["ny"], case["nz"])
    d, scalar = _DIMS[case["lattice"]], case["lattice"] == "D2Q9_D2Q5"
    rates = _uniform(g, 0.05, 0.2, 2).tolist()
    inp = dict(shape=shape, nu=rates[0], D=rates[1], omega=2.0 * math.pi / 10000.0 if case["force"] == "cos" else 0.0)
    inp["rho"] = 1.0 + _smooth(g, shape, 1, 0.01)[0]
    inp["u"] = _smooth(g, shape, d, 0.03)
    inp["phi"] = 1.0 + _smooth(g, shape, 1, 0.5)[0] if scalar else None
    if case["force"] == "uniform":
        inp["F"] = _uniform(g, 2e-6, 2e-5, d).tolist()
        inp["S"] = float(_uniform(g, 1e-6, 1e-5, 1)) if scalar else None
    else:
        inp["F"] = _smooth(g, shape, d, 2e-5)
        inp["S"] = _smooth(g, shape, 1, 1e-5)[0].contiguous() if scalar else None
    return inp


def _batch_inputs(case, seed):
    """Hartmann channels: 4..64 x 16..256 nodes (the same sizes for every seed), Ha in [0, 20], the
    Poiseuille force for U0 = 0.01."""
    g, sizes = np.random.default_rng(seed), np.random.default_rng(0)
    k = case["domains"]
    nx, ny = sizes.integers(4, 65, k), sizes.integers(16, 257, k)
    ha, nu = g.uniform(0, 20, k), g.uniform(0.02, 0.2, k)
    half = ny / 2.0
    return [(int(nx[i]), int(ny[i]), float(nu[i]), float(2 * nu[i] * 0.01 / half[i] ** 2),
             float(ha[i] ** 2 * nu[i] / half[i] ** 2)) for i in range(k)]


def _widths(case):
    w = case["width"]
    return (w, 2 * w, 2 * w, 3 * w, 3 * w, 3 * w)[:case["levels"]]


def _network_inputs(case, seed):
    g = _generator(seed)
    b, L = case["batch"], case["L"]
    cin = W.LEVEL_IN_CH if case["features"] == "levels" else W.IN_CH
    x = torch.stack([_smooth(g, (L, L, b), 1, 4.0)[0].reshape(b, L, L) for _ in range(cin)], -1)
    x = x + 0.3 * torch.randn(x.shape, generator=g, device="cuda", dtype=torch.float64)
    y = torch.stack([_smooth(g, (L, L, b), 1, 4.0)[0].reshape(b, L, L) for _ in range(W.OUT_CH)], -1)
    return x.float().contiguous(), y.float().contiguous()


def _field_inputs(case, seed):
    g = _generator(seed)
    L, b = case["L"], case["batch"]
    nu, D = _uniform(g, 0.08, 0.2, 2).tolist()
    levels = []
    for n in (L // 2, L // 4, L // 8):   # steady fields of the three coarse levels (density deviation, u, phi)
        levels.append((_smooth(g, (n, n, b), 1, 1e-4)[0], _smooth(g, (n, n, b), 2, 0.02).reshape(-1),
                       _smooth(g, (n, n, b), 1, 1.0)[0]))
    F, S = _smooth(g, (L, L, b), 2, 1e-5).reshape(-1), _smooth(g, (L, L, b), 1, 1e-4)[0].contiguous()
    y = torch.randn(b, L, L, W.OUT_CH, generator=g, device="cuda", dtype=torch.float64).float()
    return nu, D, levels, F, S, y


_FIELD_A, _FIELD_B = (0.32, 0.335, 0.337), (-0.018, -0.023, -0.023)   # about the fitted extrapolation weights
_FIELD_IN = (1e-4, 1e-4, 5e-3, 1e-6, 4e-4, 4e-4, 2e-2, 4e-6)          # r.m.s. of the level differences
_FIELD_OUT = (2e-5, 2e-5, 1e-3, 2e-7)                                 # r.m.s. of the corrections


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------

def _flow_state(case, seed):
    inp = _flow_inputs(case, seed)
    walls = tuple(a in case["walls"] for a in "xyz")
    s = Solver(case["lattice"], inp["shape"], storage=case["storage"], walls=walls, nu=inp["nu"], D_phi=inp["D"],
               residual_interval=case["interval"], flags=C.LB_FLAG_EXTERNAL_BUFFERS,
               stream=torch.cuda.current_stream().cuda_stream)
    need = C.lb_required_bytes(s.cfg)
    buffers = [torch.empty(need, dtype=torch.uint8, device="cuda") for _ in range(2)]
    C.lb_bind_buffers(s.ctx, buffers[0].data_ptr(), buffers[1].data_ptr(), need)
    if case["force"] == "uniform":
        s.set_force(*inp["F"])
        if inp["S"] is not None:
            s.set_source(inp["S"])
    else:
        F = inp["F"].contiguous()
        C.lb_set_force_field(s.ctx, F.data_ptr(), C.LB_DTYPE_F64, C.LB_MEM_DEVICE)
        if inp["S"] is not None:
            C.lb_set_source_field(s.ctx, inp["S"].data_ptr(), C.LB_DTYPE_F64, C.LB_MEM_DEVICE)
        if inp["omega"]:
            s.set_force_time(C.LB_TIME_COS, inp["omega"])
    C.lb_init_equilibrium_device(s.ctx, inp["rho"].data_ptr(), inp["u"].data_ptr(),
                                 inp["phi"].data_ptr() if inp["phi"] is not None else None)
    s.synchronize()
    info = s.info()
    q, stride = _Q[case["lattice"]], info.plane_stride
    planes = [b.view(_TORCH[case["storage"]])[:q * stride].view(q, stride)[:, :s.N] for b in buffers]
    return dict(case=case, solver=s, buffers=buffers,
                planes={b.data_ptr(): p for b, p in zip(buffers, planes)})


def _flow_run(st):
    s, case = st["solver"], st["case"]
    s.step(case["steps"])
    out = {"populations": st["planes"][s.info().buf_current]}
    if case["interval"] and case["force"] == "field" and case["lattice"] == "D2Q9_D2Q5":
        # the warm start's loop: both residuals after every block of steps
        out["residual"] = s.residual()[0]
        out["residual_scalar"] = s.residual_scalar()
    return out


def _batch_state(case, seed):
    dom = _batch_inputs(case, seed)
    cfg = C.lb_batch_config_default(storage=C.LB_STORE_F64 if case["storage"] == "f64" else C.LB_STORE_F32_DEV,
                                    check_interval=case["interval"], block=1024,
                                    stream=torch.cuda.current_stream().cuda_stream)
    h = C.lb_batch_create(cfg, dom)
    C.lb_batch_init(h)
    read = sorted(range(len(dom)), key=lambda i: dom[i][0] * dom[i][1])[::max(1, len(dom) // 4)]
    return _Batch(case, h, dom, read)


class _Batch:
    """A batch handle that is given back with its state, and the domains whose profiles are read."""

    def __init__(self, case, handle, domains, read):
        self.case, self.handle, self.domains, self.read = case, handle, domains, read

    def __del__(self):
        C.lb_batch_destroy(self.handle)


def _batch_run(b):
    C.lb_batch_run(b.handle, b.case["steps"], 1e-300)
    steps, residual, status = C.lb_batch_results(b.handle, len(b.domains))
    profiles = []
    for i in b.read:
        nx, ny = b.domains[i][:2]
        profiles.append([np.empty((ny, nx)), np.empty((2, ny, nx))])
        C.lb_batch_read_moments(b.handle, i, *profiles[-1])
    return {"steps": steps, "residual": residual, "status": status, "profiles": profiles}


class _Network:
    """A network that is given back with its state, and its device inputs and targets."""

    def __init__(self, case, seed):
        self.case = case
        self.net = W.Surrogate(L=case["L"], max_batch=case["batch"], levels=case["levels"], channels=_widths(case),
                               features=case["features"])
        self.net.init_params(seed)
        self.x, self.y = _network_inputs(case, seed)

    def __del__(self):
        self.net.close()


def _network_run(n):
    if n.case["kind"] == "forward":
        return {"y": n.net.forward(n.x)}
    loss, grad = C.lb_unet_loss_grad(n.net.h, n.x.data_ptr(), n.y.data_ptr(), n.case["batch"])
    C.lb_unet_adam(n.net.h, 1e-4)
    return {"loss": loss, "gradient": grad}


def _field_state(case, seed):
    nu, D, levels, F, S, y = _field_inputs(case, seed)
    fields = []
    for n, (rho, u, phi) in zip((case["L"] // 2, case["L"] // 4, case["L"] // 8), levels):
        f = W.Fields(n, case["batch"])
        f.rho.copy_(rho)
        f.u.copy_(u)
        f.phi.copy_(phi)
        fields.append(f)
    return dict(probs=W.Problems(case["L"], nu, D, F, S), levels=fields, y=y)


def _field_run(st):
    probs, (f1, f2, f3) = st["probs"], st["levels"]
    guess = W.guess_from_levels(f1, f2, _FIELD_A, f3, _FIELD_B)
    d1, d2 = W.level_differences(f1, f2, f3)
    x = W.features_levels(probs, d1, d2, _FIELD_IN, torch.empty(probs.B, probs.L, probs.L, W.LEVEL_IN_CH,
                                                                dtype=torch.float32, device="cuda"))
    est = W.estimate(guess, st["y"], W.CORRECTION_K2, _FIELD_OUT)
    start = W.initial_state(probs, est)
    return {"x": x, "estimate": [est.rho, est.u, est.phi], "start": [start.rho, start.u, start.phi]}


def prepare(case, seed):
    if case["family"] == "flow":
        return _flow_state(case, seed)
    if case["family"] == "batch":
        return _batch_state(case, seed)
    if case["family"] == "network":
        return _Network(case, seed)
    return _field_state(case, seed)


def run(state):
    if isinstance(state, _Batch):
        return _batch_run(state)
    if isinstance(state, _Network):
        return _network_run(state)
    return _flow_run(state) if "solver" in state else _field_run(state)


# ---------------------------------------------------------------------------
# work
# ---------------------------------------------------------------------------

def _layers(case):
    """(side, inputs, outputs) of every convolution, in parameter order."""
    c, L = _widths(case), case["L"]
    cin = W.LEVEL_IN_CH if case["features"] == "levels" else W.IN_CH
    out = []
    for l in range(case["levels"]):
        out += [(L >> l, cin if l == 0 else c[l - 1], c[l]), (L >> l, c[l], c[l])]
    out += [(L >> l, c[l] + c[l + 1], c[l]) for l in range(case["levels"] - 2, -1, -1)]
    return out + [(L, c[0], W.OUT_CH)]


def work(case):
    if case["family"] == "flow":
        n = case["nx"] * case["ny"] * case["nz"]
        d, scalar = _DIMS[case["lattice"]], case["lattice"] == "D2Q9_D2Q5"
        state = 2 * n * _Q[case["lattice"]] * _ELEM[case["storage"]]
        field = n * (d + scalar) * max(4, _ELEM[case["storage"]]) if case["force"] != "uniform" else 0
        # every step reads the state that the step before wrote, unless it fits on the chip
        passes = 1 if state <= _ON_CHIP else case["steps"]
        return {"bytes": passes * (state + field), "flops": case["steps"] * n * _NODE_FLOPS[case["lattice"]]}
    if case["family"] == "batch":
        # the sizes' means: 34 x 136 nodes a domain; domains stay in the cache or in LDS
        n = case["domains"] * 34 * 136
        return {"bytes": 2 * 9 * n * _ELEM[case["storage"]], "flops": case["steps"] * n * _NODE_FLOPS["D2Q9"]}
    if case["family"] == "network":
        layers, b = _layers(case), case["batch"]
        flops = sum(18.0 * b * s * s * ci * co for s, ci, co in layers)
        params = sum(9 * ci * co + co for _, ci, co in layers)
        px = b * case["L"] ** 2
        ends = 4 * px * (layers[0][1] + W.OUT_CH)
        if case["kind"] == "forward":
            return {"bytes": ends + 2 * params, "flops": flops}
        # training keeps every activation for the gradient (bf16, written once and read once), reads the
        # target and updates parameters and both Adam moments
        acts = sum(2 * 2 * b * s * s * co for s, _, co in layers[:-1])
        return {"bytes": ends + 4 * px * W.OUT_CH + acts + 4 * 7 * params, "flops": 3.0 * flops}
    n = case["batch"] * case["L"] ** 2
    coarse = 4 * 8 * n * (1 / 4 + 1 / 16 + 1 / 64)
    # coarse fields, force, source and network output in; network input, estimate and start state out
    return {"bytes": coarse + 3 * 8 * n + 4 * 4 * n + 4 * W.LEVEL_IN_CH * n + 2 * 4 * 8 * n, "flops": 400 * n}


# ---------------------------------------------------------------------------
# the same outputs from plain float64 torch
# ---------------------------------------------------------------------------

_D2Q9 = [(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)]
_D2Q5 = _D2Q9[:5]
_DIGIT = {0: 0, 1: 1, -1: 2}


def _velocities(lattice):
    if lattice == "D3Q27":
        v = (0, 1, -1)
        return [(v[a % 3], v[a // 3 % 3], v[a // 9]) for a in range(27)]
    return [e + (0,) for e in _D2Q9]


def _pull_table(e, shape, walls):
    """Flat index into [Q][N] that population a of node x comes from: a at x - e, or at a wall the
    opposite population of x itself (halfway bounce-back)."""
    c = [torch.arange(n, device="cuda") for n in shape]
    z, y, x = torch.meshgrid(c[2], c[1], c[0], indexing="ij")
    pos, n = (x.reshape(-1), y.reshape(-1), z.reshape(-1)), shape[0] * shape[1] * shape[2]
    node = torch.arange(n, device="cuda")
    table = torch.empty(len(e), n, dtype=torch.int64, device="cuda")
    for a, ea in enumerate(e):
        blocked = torch.zeros(n, dtype=torch.bool, device="cuda")
        src = []
        for i in range(3):
            p = pos[i] - ea[i]
            if walls[i]:
                blocked |= (p < 0) | (p >= shape[i])
            src.append(p % shape[i])
        flat = src[0] + shape[0] * (src[1] + shape[1] * src[2])
        opposite = e.index(tuple(-v for v in ea))
        table[a] = torch.where(blocked, opposite * n + node, a * n + flat)
    return table


_RAW = ((1.0, 1.0, 1.0), (0.0, 1.0, -1.0), (0.0, 1.0, 1.0))       # moments 0, 1, 2 of velocities 0, +1, -1
_BACK = ((1.0, 0.0, -1.0), (0.0, 0.5, 0.5), (0.0, -0.5, 0.5))     # and back


def _each_axis(m, d, fn):
    """fn on the three entries along every digit axis of m [3]*d + [N]."""
    for a in range(d):
        m = torch.stack(fn(a, *m.unbind(a)), a)
    return m


def _linear(rows):
    return lambda a, *v: [sum(r[i] * v[i] for i in range(3) if r[i]) for r in rows]


def _about(u):
    return lambda a, k0, k1, k2: [k0, k1 - u[a] * k0, k2 - 2 * u[a] * k1 + u[a] * u[a] * k0]


def _collide(f, e, d, nu, fpre, ftot, lorentz=None):
    """Cascaded collision with both half force steps of [Q][N] populations: (f, rho, u), all other rates 1.
    Raw moments, first-order ones from the half-forced velocity, central moments about it, relaxation to
    rho prod(1, 0, 1/3), and back; then the first-order change F_tot . e / <e_x|e_x>."""
    n = f.shape[1]
    order = [sum(_DIGIT[ea[i]] * 3 ** (d - 1 - i) for i in range(d)) for ea in e]
    grid = torch.empty_like(f)
    grid[order] = f
    m = _each_axis(grid.view(*([3] * d), n), d, _linear(_RAW))
    zero = (0,) * d
    unit = [tuple(1 if i == a else 0 for i in range(d)) for a in range(d)]
    twos = [tuple(2 if i == a else 0 for i in range(d)) for a in range(d)]
    rho = m[zero]
    fpre, ftot = list(fpre), list(ftot)
    if lorentz is not None:   # implicit midpoint of the velocity-dependent force -s u_x
        ux = (m[unit[0]] + 0.5 * fpre[0]) / (rho + 0.5 * lorentz)
        fpre[0], ftot[0] = fpre[0] - lorentz * ux, ftot[0] - lorentz * ux
    u = [(m[unit[a]] + 0.5 * fpre[a]) / rho for a in range(d)]
    k = m.clone()
    for a in range(d):
        k[unit[a]] = rho * u[a]
    k = _each_axis(k, d, _about(u))
    change = torch.zeros_like(k)
    shear = 1.0 / (3.0 * nu + 0.5)
    for idx in np.ndindex(*([3] * d)):
        if sum(idx) < 2:
            continue
        rest = 1.0
        for p in idx:
            rest *= (1.0, 0.0, 1.0 / 3.0)[p]
        change[idx] = k[idx] - rho * rest
        if sum(idx) == 2 and 2 not in idx:
            change[idx] = shear * change[idx]
    mean = sum(change[t] for t in twos) / d
    for t in twos:
        change[t] = mean + shear * (change[t] - mean)
    m = m - _each_axis(change, d, _about([-v for v in u]))
    f = _each_axis(m, d, _linear(_BACK)).reshape(3 ** d, n)[order]
    norm = 6.0 if d == 2 else 18.0
    for a, ea in enumerate(e):
        for i in range(d):
            if ea[i]:
                f[a] += ea[i] * ftot[i] / norm
    return f, rho, u


def _collide_scalar(g, u, spre, stot, D):
    """D2Q5 collision with both half source steps: first central moments relax with the diffusivity's
    rate, second ones to phi / 3."""
    phi = g.sum(0) + 0.5 * spre
    w = 1.0 / (3.0 * D + 0.5)
    g = g.clone()
    removed_first, removed_second = [], []
    for a in range(2):
        p, q = g[1 + a], g[3 + a]
        first, second = p - q, p + q
        c1 = w * (first - u[a] * phi)
        c2 = second - 2 * u[a] * first + u[a] ** 2 * phi - phi / 3.0
        removed_first.append(c1)
        removed_second.append(c2 + 2 * u[a] * c1)
    g[0] += sum(removed_second)
    for a in range(2):
        g[1 + a] -= 0.5 * (removed_second[a] + removed_first[a])
        g[3 + a] -= 0.5 * (removed_second[a] - removed_first[a])
    return g + 0.2 * stot


def _equilibrium(e, d, rho, u):
    f = []
    for ea in e:
        v = rho
        for i in range(d):
            v = v * (2.0 / 3.0 - u[i] ** 2 if ea[i] == 0 else 0.5 * (1.0 / 3.0 + u[i] ** 2 + ea[i] * u[i]))
        f.append(v)
    return torch.stack(f)


def _weights(e, d):
    return torch.tensor([math.prod(2.0 / 3.0 if v == 0 else 1.0 / 6.0 for v in ea[:d]) for ea in e],
                        dtype=torch.float64, device="cuda")


def _flow_exact(case, seed):
    inp = _flow_inputs(case, seed)
    d, e, shape = _DIMS[case["lattice"]], _velocities(case["lattice"]), inp["shape"]
    walls = ["x" in case["walls"], "y" in case["walls"], "z" in case["walls"] and d == 3]
    f = _equilibrium(e, d, inp["rho"], inp["u"])
    table = _pull_table(e, shape, walls)
    g = gtable = None
    if inp["phi"] is not None:
        u, phi = inp["u"], inp["phi"]
        g = torch.stack([phi * (1.0 / 3.0 - u[0] ** 2 - u[1] ** 2)] +
                        [0.5 * phi * (1.0 / 3.0 + u[i] ** 2 + s * u[i]) for s in (1, -1) for i in (0, 1)])
        gtable = _pull_table([v + (0,) for v in _D2Q5], shape, walls)
    for step in range(case["steps"]):
        tau = [math.cos(inp["omega"] * (step + h)) for h in (0.0, 0.5, 1.0)]
        pre, post = 0.5 * (tau[0] + tau[1]), 0.5 * (tau[1] + tau[2])
        f = f.reshape(-1)[table]
        F = inp["F"]
        f, _, u = _collide(f, e, d, inp["nu"], [pre * F[i] for i in range(d)],
                           [0.5 * (pre + post) * F[i] for i in range(d)])
        if g is not None:
            g = _collide_scalar(g.reshape(-1)[gtable], u, inp["S"], inp["S"], inp["D"])
    f = f - _weights(e, d)[:, None]
    out = {"populations": f if g is None else torch.cat([f, g])}
    if case["interval"] and case["force"] == "field" and case["lattice"] == "D2Q9_D2Q5":
        out.update(residual=None, residual_scalar=None)
    return out


def _batch_exact(case, seed):
    dom = _batch_inputs(case, seed)
    read = sorted(range(len(dom)), key=lambda i: dom[i][0] * dom[i][1])[::max(1, len(dom) // 4)]
    e = _velocities("D2Q9")
    profiles = []
    for i in read:
        nx, ny, nu, force, s = dom[i]
        f = _weights(e, 2)[:, None].repeat(1, nx * ny)
        table = _pull_table(e, (nx, ny, 1), (False, True, False))
        for _ in range(case["steps"]):
            f, _, _ = _collide(f.reshape(-1)[table], e, 2, nu, [force, 0.0], [force, 0.0], lorentz=s)
        f = f.reshape(-1)[table]
        rho = f.sum(0)
        jx = sum(ea[0] * f[a] for a, ea in enumerate(e) if ea[0])
        jy = sum(ea[1] * f[a] for a, ea in enumerate(e) if ea[1])
        u = torch.stack([(jx + 0.5 * force) / (rho + 0.5 * s), jy / rho])
        profiles.append([rho.view(ny, nx).cpu().numpy(), u.view(2, ny, nx).cpu().numpy()])
    return {"steps": None, "residual": None, "status": None, "profiles": profiles}


def _conv(x, w, b):
    """Circular 3 x 3 convolution of [B][H][W][Ci] with [Co][9][Ci] weights as nine shifted products."""
    shape = x.shape[:3] + (w.shape[0],)
    out = b.expand(shape).reshape(-1, w.shape[0])
    for tap in range(9):
        shifted = torch.roll(x, (1 - tap // 3, 1 - tap % 3), (1, 2))
        out = out + shifted.reshape(-1, x.shape[3]) @ w[:, tap].t().contiguous()
    return out.view(shape)


def _network_exact(case, seed):
    x, y = (t.double() for t in _network_inputs(case, seed))
    g = np.random.default_rng(seed)   # the draws of Surrogate.init_params
    params = []
    for _, ci, co in _layers(case):
        std = math.sqrt(2.0 / (9 * ci))
        w = (g.standard_normal(co * 9 * ci) * std).astype(np.float32)
        params += [torch.from_numpy(w).double().cuda().view(co, 9, ci), torch.zeros(co, dtype=torch.float64, device="cuda")]
    train = case["kind"] == "train"
    for p in params:
        p.requires_grad_(train)
    layers = [(params[2 * i], params[2 * i + 1]) for i in range(len(params) // 2)]
    n, skips, h = case["levels"], [], x
    with torch.set_grad_enabled(train):
        for l in range(n):
            h = _conv(_conv(h, *layers[2 * l]).relu(), *layers[2 * l + 1]).relu()
            if l < n - 1:
                skips.append(h)
                b, s = h.shape[0], h.shape[1] // 2
                h = h.view(b, s, 2, s, 2, h.shape[3]).mean((2, 4))
        for l in range(n - 2, -1, -1):
            up = h.repeat_interleave(2, 1).repeat_interleave(2, 2)
            h = _conv(torch.cat([skips[l], up], 3), *layers[2 * n + n - 2 - l]).relu()
        out = _conv(h, *layers[-1])
        if not train:
            return {"y": out}
        loss = ((out - y) ** 2).mean()
        loss.backward()
    return {"loss": float(loss.detach()), "gradient": torch.cat([p.grad.reshape(-1) for p in params])}


def _prolonged(a, scale):
    """Periodic Catmull-Rom interpolation of [planes][L][L] to twice the size, times scale."""
    even, odd = (-0.0234375, 0.2265625, 0.8671875, -0.0703125), (-0.0703125, 0.8671875, 0.2265625, -0.0234375)
    for dim in (1, 2):
        lo = sum(w * torch.roll(a, 2 - i, dim) for i, w in enumerate(even))   # taps X-2 .. X+1
        hi = sum(w * torch.roll(a, 1 - i, dim) for i, w in enumerate(odd))    # taps X-1 .. X+2
        shape = list(a.shape)
        shape[dim] *= 2
        a = torch.stack([lo, hi], dim + 1).reshape(shape)
    return scale * a


def _projected(a, k2max=0):
    """[planes][L][L] without mean, Nyquist lines and the modes 0 < |k|^2 <= k2max."""
    L = a.shape[1]
    s = torch.fft.fft2(a)
    k = torch.fft.fftfreq(L, 1.0 / L, device="cuda", dtype=torch.float64)
    k2 = k[:, None] ** 2 + k[None, :] ** 2
    keep = (k2 > k2max) & (k[:, None].abs() < L // 2) & (k[None, :].abs() < L // 2)
    return torch.fft.ifft2(s * keep).real


def _field_exact(case, seed):
    nu, D, levels, F, S, y = _field_inputs(case, seed)
    L, b = case["L"], case["batch"]
    scale = (0.25, 0.5, 1.0)
    f1, f2, f3 = ([t.view(-1, n, n) for t in lev] for lev, n in zip(levels, (L // 2, L // 4, L // 8)))
    up = lambda f: [_prolonged(t, s) for t, s in zip(f, scale)]
    p2, p3 = up(f2), up(up(f3))
    guess = [_projected(t) for t in up([(1 + wa) * h - wa * q + wb * (q - o) for h, q, o, wa, wb in
                                        zip(f1, p2, p3, _FIELD_A, _FIELD_B)])]
    d1 = [_projected(t) for t in up([h - q for h, q in zip(f1, p2)])]
    d2 = [_projected(t) for t in up(up([q - o for q, o in zip(f2, up(f3))]))]
    F, S = F.view(2, b, L, L), S.view(b, L, L)
    one = torch.ones_like(S)
    fs = 1.0 / (nu * W.K0 ** 2 * W.U0)
    ch = [fs * F[0], fs * F[1], S / (D * W.K0 ** 2 * W.PHI0), one * (nu - W.RATE_MID) / W.RATE_HALF,
          one * (D - W.RATE_MID) / W.RATE_HALF]
    for d, sc in ((d1, _FIELD_IN[:4]), (d2, _FIELD_IN[4:])):
        u = d[1].view(2, b, L, L)
        ch += [u[0] / sc[0], u[1] / sc[1], d[2] / sc[2], d[0] / sc[3]]
    corr = [_projected(_FIELD_OUT[c] * y[..., c].double(), W.CORRECTION_K2) for c in range(4)]
    u = guess[1].view(2, b, L, L) + torch.stack([corr[0], corr[1]])
    phi, rho = guess[2] + corr[2], guess[0] + corr[3]
    full = 1.0 + rho
    shift = (full * u).sum((2, 3), keepdim=True) / full.sum((1, 2))[None, :, None, None]
    start = [full, u - shift - F / (2.0 * full), phi - 0.5 * S]
    flat = lambda v: [t.reshape(-1) for t in v]
    return {"x": torch.stack(ch, 3), "estimate": flat([rho, u, phi]), "start": flat(start)}


def exact(case, seed):
    if case["family"] == "flow":
        # gathers over all populations of every step: about 3e8 node updates fit in the time
        if case["nx"] * case["ny"] * case["nz"] * case["steps"] > 3e8:
            return None
        return _flow_exact(case, seed)
    return {"batch": _batch_exact, "network": _network_exact, "fields": _field_exact}[case["family"]](case, seed)
