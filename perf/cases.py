"""Workloads of the stencil library, for timing it over the range of its use.

A case names one way a program uses the library through its Python binding:

  sweep     time loops of one plan: 2D and 3D heat and second-order wave, any
            storage type and space order, sources and receivers on or off the
            grid, an absorbing layer, zero or periodic halo.  The plan is tuned
            once, as the benchmark and the tests of this repository do, and the
            loop is restarted from the same levels on every pass.
  batch     independent shots of uneven size in one call.
  gradient  the misfit and its gradient of one shot, with checkpoints.
  program   one fused evaluation of the PW advection program.
  rank      one rank's part of a decomposed run: per step the boundary slabs,
            the packed faces, the interior box and the unpacked halos.  Its own
            faces stand in for the neighbours'.

`listed` holds the fixed cases, `draw` gives others of the same ranges, `exact`
evaluates a case in 64 bits with plain torch operations.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2404_02218_amd as S
from paper_2404_02218_amd.program import Program, pw_advection_terms

DEVICE = "cuda"
STORAGE = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
H = 10.0        # grid spacing, m
ALPHA = 0.05    # a dt / h^2 of the heat sweeps (stable for every space order in 3D)


def listed():
    """The fixed cases."""
    return [
        # the smallest call: a 2D field that fits in cache, bound by launches
        _sweep("heat2d_256_so2", "heat", (256, 256), 2, 100),
        # the paper's 2D size (8192^2) at its highest space order: one shot
        _sweep("wave2d_8192_so8", "wave", (8192, 8192), 8, 32, nsrc=1, nrec=64),
        # the headline: a 3D shot of 512^3
        _sweep("wave3d_512_so8", "wave", (512, 512, 512), 8, 48, nsrc=1),
        # the same sweep with fields stored in bfloat16
        _sweep("wave3d_512_so8_bf16", "wave", (512, 512, 512), 8, 24, nsrc=1, dtype="bf16"),
        # a ragged half-precision model with a receiver line
        _sweep("wave3d_ragged_so8_f16", "wave", (207, 301, 259), 8, 24, nsrc=2, nrec=64, dtype="f16"),
        # the paper's 3D heat size, space order 4
        _sweep("heat3d_512_so4", "heat", (512, 512, 512), 4, 40),
        # a small 3D model, run many times in a study: bound by latency
        _sweep("wave3d_small_so8", "wave", (61, 75, 90), 8, 200, nsrc=1, nrec=16),
        # a shot with an absorbing layer and source and receivers off the grid
        _sweep("wave3d_256_absorbing", "wave", (256, 256, 256), 8, 60, nsrc=1, nrec=64, layer=32, offgrid=True),
        # uneven shots of a survey, in one call
        {"name": "batch_8_shots", "path": "batch", "shots": 8, "smallest": 96, "largest": 224, "steps": 50},
        # one gradient of an inversion: forward, adjoint, imaging
        {"name": "gradient_128", "path": "gradient", "nz": 128, "ny": 128, "nx": 128, "steps": 100, "every": 25,
         "nrec": 64},
        # PW advection of three velocity components
        {"name": "pw_advection_384", "path": "program", "nz": 384, "ny": 384, "nx": 384},
        # one of 8 ranks of the 512^3 model, split along z
        {"name": "rank_64x512x512", "path": "rank", "nz": 64, "ny": 512, "nx": 512, "steps": 8, "dtype": "f32"},
    ]


def _sweep(name, kind, shape, order, steps, nsrc=0, nrec=0, dtype="f32", layer=0, offgrid=False, periodic=False):
    c = {"name": name, "path": "sweep", "kind": kind, "order": order, "steps": steps, "nsrc": nsrc, "nrec": nrec,
         "dtype": dtype, "layer": layer, "offgrid": offgrid, "periodic": periodic}
    c.update(zip(("nz", "ny", "nx")[3 - len(shape):], shape))
    return c


def draw(rng: random.Random):
    """One more case of the same ranges."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    path = rng.choices(("sweep3", "sweep2", "batch", "gradient", "program", "rank"), (6, 4, 2, 2, 1, 2))[0]
    if path == "sweep3":
        kind = rng.choice(("wave", "wave", "heat"))
        dtype = rng.choice(("f32", "f32", "bf16", "f16"))
        order = 8 if kind == "wave" and rng.random() < 0.75 else rng.choice((2, 4, 8))
        periodic = rng.random() < 0.15
        layer = rng.choice((8, 16, 24)) if kind == "wave" and dtype == "f32" and rng.random() < 0.25 else 0
        points = kind == "wave"
        c = _sweep("", kind, [size(40, 400) for _ in range(3)], order, rng.randint(10, 40),
                   nsrc=rng.randint(1, 4) if points else 0, nrec=rng.choice((0, 16, 64)) if points else 0, dtype=dtype,
                   layer=layer, offgrid=points and rng.random() < 0.25, periodic=periodic)
    elif path == "sweep2":
        kind = rng.choice(("wave", "heat"))
        points = kind == "wave"
        c = _sweep("", kind, [size(120, 6000) for _ in range(2)], rng.choice((2, 4, 8)), rng.randint(10, 60),
                   nsrc=rng.randint(1, 4) if points else 0, nrec=rng.choice((0, 16, 64)) if points else 0,
                   dtype=rng.choice(("f32", "f32", "f32", "bf16", "f16")), offgrid=points and rng.random() < 0.25)
        if kind == "wave" and c["dtype"] == "f32" and rng.random() < 0.25:
            c["layer"] = rng.choice((8, 16, 24))
    elif path == "batch":
        lo = size(48, 120)
        c = {"path": "batch", "shots": rng.randint(2, 10), "smallest": lo, "largest": size(lo + 1, 230),
             "steps": rng.randint(10, 50)}
    elif path == "gradient":
        every = rng.randint(5, 25)
        c = {"path": "gradient", "steps": rng.randint(30, 100), "every": every, "nrec": rng.choice((16, 64)),
             "nz": size(40, 140), "ny": size(40, 140), "nx": size(40, 140)}
    elif path == "program":
        c = {"path": "program", "nz": size(48, 384), "ny": size(48, 384), "nx": size(48, 384)}
    else:
        c = {"path": "rank", "nz": size(24, 96), "ny": size(96, 512), "nx": size(96, 512), "steps": rng.randint(2, 8),
             "dtype": rng.choice(("f32", "f32", "bf16", "f16"))}
    c.pop("name", None)
    return c


# ------------------------------------------------------------------ inputs

def _shape(case):
    return tuple(case[k] for k in ("nz", "ny", "nx") if k in case)


def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed))


def _layered_velocity(shape, g):
    """Eight layers of 1.5 to 4.5 km/s along the first axis, with 5% noise."""
    v = 1500.0 + 3000.0 / 7.0 * (torch.arange(shape[0], device=DEVICE, dtype=torch.float64) * 8 // shape[0]).clamp(max=7)
    noise = torch.rand(shape, generator=g, device=DEVICE, dtype=torch.float32)
    return v.reshape([-1] + [1] * (len(shape) - 1)) * (0.95 + 0.1 * noise.double())


def _dt(order, ndim, vmax):
    """Half the leapfrog limit of the centred star of this order."""
    c = S.second_derivative_weights(order)
    symbol = -(c[0] + 2 * sum(ck * (-1) ** (k + 1) for k, ck in enumerate(c[1:])))
    return H / (vmax * math.sqrt(ndim * symbol))


def _wavefield(shape, g):
    """A band-limited random level: the wave in the middle of a run."""
    u = torch.randn(shape, generator=g, device=DEVICE, dtype=torch.float32)[None, None]
    pool = torch.nn.functional.avg_pool3d if len(shape) == 3 else torch.nn.functional.avg_pool2d
    for _ in range(2):
        u = pool(u, 3, stride=1, padding=1)
    return u[0, 0]


def _ricker(n, dt, f0=20.0):
    a = (math.pi * f0 * (np.arange(n) * dt - 1.0 / f0)) ** 2
    return (1.0 - 2.0 * a) * np.exp(-a)


def _points(shape, n, rng, offgrid):
    if n == 0:
        return None
    p = np.stack([rng.integers(1, s - 2, size=n) for s in shape], axis=1)
    return p + rng.random(p.shape) if offgrid else p


def _inner(field, halo):
    return field.view[tuple(slice(halo, s - halo) for s in field.view.shape)]


def _start(plan, level):
    """A field of the plan that holds this level; its storage is what a run restarts from."""
    f = plan.field()
    _inner(f, plan.halo).copy_(level)
    return f


def _profiles(shape, width):
    return [S.damping_profile(n, width, 0.1) for n in shape]


def _sweep_inputs(case, seed):
    """Levels, coefficients and points of a sweep; levels and beta as the storage type holds them."""
    shape, g, rng = _shape(case), _generator(seed), np.random.default_rng(seed)
    store = STORAGE[case["dtype"]]
    x = {"shape": shape, "radius": case["order"] // 2}
    if case["kind"] == "heat":
        x["coeffs"] = S.heat_weights(case["order"], ALPHA)
        x["u"] = torch.rand(shape, generator=g, device=DEVICE, dtype=torch.float32).to(store)
        return x
    x["coeffs"] = S.second_derivative_weights(case["order"])
    v = _layered_velocity(shape, g)
    dt = _dt(case["order"], len(shape), 4725.0)
    x["beta"] = ((dt / H) ** 2 * v * v).to(store)
    u = _wavefield(shape, g)
    x["prev"] = (u + 0.1 * _wavefield(shape, g)).to(store)
    x["u"] = u.to(store)
    x["src"] = _points(shape, case["nsrc"], rng, case["offgrid"])
    x["rec"] = _points(shape, case["nrec"], rng, case["offgrid"])
    amp = 5.0 * _ricker(case["steps"], dt).reshape(-1, 1) * rng.uniform(0.5, 1.5, size=(1, case["nsrc"]))
    x["amp"] = torch.from_numpy(np.ascontiguousarray(amp)).to(DEVICE)
    return x


def _shot_shapes(case, seed):
    """Cubes of seeded uneven sizes; the largest and the smallest are always there."""
    rng = np.random.default_rng(case["shots"] * 1000 + case["largest"])
    n = rng.integers(case["smallest"], case["largest"] + 1, size=case["shots"])
    n[0], n[1] = case["largest"], case["smallest"]
    return [(int(k),) * 3 for k in n]


def _shot_case(case, shape):
    return _sweep("", "wave", shape, 8, case["steps"], nsrc=1)


def _gradient_inputs(case, seed):
    shape, g, rng = _shape(case), _generator(seed), np.random.default_rng(seed)
    v = _layered_velocity(shape, g)
    dt = _dt(8, 3, 4725.0)
    y, x = shape[1] // 2, shape[2]
    rec = np.array([[6, y, int(round(4 + j * (x - 9) / (case["nrec"] - 1)))] for j in range(case["nrec"])])
    wavelet = torch.from_numpy(_ricker(case["steps"], dt, 25.0).reshape(-1, 1)).to(DEVICE)
    # data of the size the shot itself records at its receivers
    d_obs = 1e-3 * torch.from_numpy(rng.standard_normal((case["steps"], case["nrec"]))).to(DEVICE)
    return {"shape": shape, "m": 1.0 / (v * v), "dt": dt, "src": np.array([[6, y, x // 2]]), "rec": rec,
            "wavelet": wavelet, "d_obs": d_obs}


def _velocities(shape, seed):
    """Three velocity components with a halo of one, wrapped around."""
    g = _generator(seed)
    return [torch.nn.functional.pad(torch.randn(shape, generator=g, device=DEVICE)[None, None], (1,) * 6,
                                    mode="circular")[0, 0] for _ in range(3)]


# ----------------------------------------------------------------- prepare

def prepare(case, seed):
    """Plan, fields and inputs that a program has in hand before the call."""
    return {"sweep": _prepare_sweep, "batch": _prepare_batch, "gradient": _prepare_gradient,
            "program": _prepare_program, "rank": _prepare_rank}[case["path"]](case, seed)


def _prepare_sweep(case, seed):
    x = _sweep_inputs(case, seed)
    wave = case["kind"] == "wave"
    plan = S.Plan(S.WAVE2 if wave else S.HEAT, x["shape"], x["radius"], x["coeffs"], dtype=S.DTYPES[case["dtype"]],
                  bc=S.BC_PERIODIC if case["periodic"] else S.BC_DIRICHLET0)
    if case["layer"]:
        plan.set_damping(_profiles(x["shape"], case["layer"]))
    starts = [_start(plan, x["u"])] + ([_start(plan, x["prev"])] if wave else [])
    fields = [_start(plan, x["u"]), _start(plan, x["prev"] if wave else x["u"])]
    st = {"case": case, "plan": plan, "starts": starts}
    if wave:
        fields.append(_start(plan, x["beta"]))
        st.update(src=x["src"], rec=x["rec"], amp=x["amp"])
        if x["rec"] is not None:
            st["trace"] = torch.zeros((case["steps"], case["nrec"]), dtype=torch.float64, device=DEVICE)
    st["fields"] = fields
    plan.tune(fields)
    return st


def _prepare_batch(case, seed):
    shapes = _shot_shapes(case, seed)
    plan = S.BatchPlan(shapes, 4, S.second_derivative_weights(8))
    shots = [_sweep_inputs(_shot_case(case, s), seed + 7919 * i) for i, s in enumerate(shapes)]
    fields, starts = [], []
    for i, x in enumerate(shots):
        f = [plan.field(i) for _ in range(3)]
        for k, name in enumerate(("u", "prev", "beta")):
            _inner(f[k], plan.halo).copy_(x[name])
        fields.append(f)
        starts.append([f[0].storage.clone(), f[1].storage.clone()])
    plan.tune(fields)
    return {"case": case, "plan": plan, "fields": fields, "starts": starts, "src": [x["src"] for x in shots],
            "amp": [x["amp"] for x in shots]}


def _prepare_gradient(case, seed):
    x = _gradient_inputs(case, seed)
    plan = S.Plan(S.WAVE2, x["shape"], 4, S.second_derivative_weights(8))
    fields = [plan.field() for _ in range(3)]
    plan.wave_beta(x["m"], x["dt"], H, fields[2])
    plan.tune(fields)
    nbytes = plan.adjoint_workspace_bytes(case["steps"], case["every"])
    return {"case": case, "plan": plan, "fields": fields, "x": x,
            "workspace": torch.empty(nbytes, dtype=torch.uint8, device=DEVICE),
            "trace": torch.zeros((case["steps"], case["nrec"]), dtype=torch.float64, device=DEVICE),
            "misfit": torch.zeros(1, dtype=torch.float64, device=DEVICE),
            "grad": torch.zeros(x["shape"], dtype=torch.float64, device=DEVICE)}


def _prepare_program(case, seed):
    shape = _shape(case)
    plan = Program(shape, 1, 3, 3, pw_advection_terms(1.0, 1.0, 1.0))
    ins, outs = [plan.field() for _ in range(3)], [plan.field() for _ in range(3)]
    for f, v in zip(ins, _velocities(shape, seed)):
        f.view.copy_(v)
    plan.tune(ins + outs)
    return {"case": case, "plan": plan, "ins": ins, "outs": outs}


def _prepare_rank(case, seed):
    x = _sweep_inputs(_sweep("", "wave", _shape(case), 8, case["steps"], dtype=case["dtype"]), seed)
    plan = S.Plan(S.WAVE2, x["shape"], 4, x["coeffs"], dtype=S.DTYPES[case["dtype"]])
    faces = plan.exchanges([8, 1, 1], [3, 0, 0])
    nz, ny, nx = x["shape"]
    starts = [_start(plan, x["u"]), _start(plan, x["prev"])]
    buf = torch.empty(plan.exchange_elems(faces), dtype=STORAGE[case["dtype"]], device=DEVICE)
    for f in starts:
        plan.pack(f, faces, buf)
        plan.unpack(f, faces, buf)
    return {"case": case, "plan": plan, "starts": starts, "beta": _start(plan, x["beta"]), "faces": faces, "buf": buf,
            "fields": [plan.field(), plan.field()],
            "edges": [([0, 0, 0], [4, ny, nx]), ([nz - 4, 0, 0], [nz, ny, nx])],
            "middle": ([4, 0, 0], [nz - 4, ny, nx])}


# --------------------------------------------------------------------- run

def run(state):
    """One pass; its outputs."""
    return {"sweep": _run_sweep, "batch": _run_batch, "gradient": _run_gradient, "program": _run_program,
            "rank": _run_rank}[state["case"]["path"]](state)


def _run_sweep(st):
    case, plan, f = st["case"], st["plan"], list(st["fields"])
    for field, start in zip(f, st["starts"]):
        field.storage.copy_(start.storage)
    if case["kind"] == "heat":
        plan.run(f, case["steps"])
        return {"u": _inner(f[0], plan.halo)}
    out = {}
    (plan.run_interp if case["offgrid"] else plan.run)(f, case["steps"], src=st["src"], src_amp=st["amp"],
                                                       rec=st["rec"], rec_trace=st.get("trace"))
    if "trace" in st:
        out["trace"] = st["trace"]
    out["u"], out["prev"] = _inner(f[0], plan.halo), _inner(f[1], plan.halo)
    return out


def _run_batch(st):
    f = [list(shot) for shot in st["fields"]]
    for shot, start in zip(f, st["starts"]):
        shot[0].storage.copy_(start[0])
        shot[1].storage.copy_(start[1])
    st["plan"].run(f, st["case"]["steps"], srcs=st["src"], src_amps=st["amp"])
    return [[_inner(shot[0], 4), _inner(shot[1], 4)] for shot in f]


def _run_gradient(st):
    x, case = st["x"], st["case"]
    st["plan"].gradient(list(st["fields"]), x["m"], x["dt"], H, case["steps"], case["every"], st["workspace"], x["src"],
                        x["wavelet"], x["rec"], st["trace"], x["d_obs"], st["misfit"], st["grad"])
    return {"misfit": st["misfit"], "grad": st["grad"], "trace": st["trace"]}


def _run_program(st):
    st["plan"].apply_program(st["outs"], st["ins"])
    return [_inner(f, 1) for f in st["outs"]]


def _run_rank(st):
    plan, (cur, prev), beta = st["plan"], st["fields"], st["beta"]
    cur.storage.copy_(st["starts"][0].storage)
    prev.storage.copy_(st["starts"][1].storage)
    for _ in range(st["case"]["steps"]):
        # the new level overwrites the previous one in place
        for lo, hi in st["edges"]:
            plan.apply(prev, [cur, prev, beta], lo, hi)
        plan.pack(prev, st["faces"], st["buf"])
        lo, hi = st["middle"]
        plan.apply(prev, [cur, prev, beta], lo, hi)
        plan.unpack(prev, st["faces"], st["buf"])
        cur, prev = prev, cur
    return {"u": _inner(cur, plan.halo), "prev": _inner(prev, plan.halo)}


# -------------------------------------------------------------------- work

def work(case):
    """Bytes and operations of one pass: per step each level and coefficient read once and the new level
    written once, and the additions and multiplications of the star (symmetric taps added first)."""
    path = case["path"]
    size = {"f32": 4}.get(case.get("dtype", "f32"), 2)
    if path == "batch":
        pts = sum(s[0] ** 3 for s in _shot_shapes(case, 0)) * case["steps"]
        return {"bytes": 16 * pts, "flops": 40 * pts}
    pts = math.prod(_shape(case))
    if path == "program":
        return {"bytes": 24 * pts, "flops": 60 * 3 * pts}
    steps = case["steps"]
    if path == "gradient":
        # forward and backward sweeps; the forward levels again; 8 bytes of gradient
        return {"bytes": (16 + 16 + 12) * pts * steps + 24 * pts, "flops": 3 * 40 * pts * steps}
    ndim = len(_shape(case))
    if path == "rank":
        return {"bytes": 4 * size * pts * steps, "flops": 40 * pts * steps}
    star = 1 + 3 * ndim * (case["order"] // 2)
    wave = case["kind"] == "wave"
    return {"bytes": (4 if wave else 2) * size * pts * steps, "flops": (star + (4 if wave else 1)) * pts * steps}


# ------------------------------------------------------------------- exact

def exact(case, seed):
    """The outputs of run() in 64 bits, with plain torch operations."""
    return {"sweep": _exact_sweep, "batch": _exact_batch, "gradient": _exact_gradient, "program": _exact_program,
            "rank": _exact_rank}[case["path"]](case, seed)


def _shifted(padded, halo, axis, k):
    return padded[tuple(slice(halo + (k if d == axis else 0), n - halo + (k if d == axis else 0))
                        for d, n in enumerate(padded.shape))]


def _star(padded, halo, coeffs):
    nd = padded.dim()
    acc = nd * coeffs[0] * _shifted(padded, halo, 0, 0)
    for axis in range(nd):
        for k, c in enumerate(coeffs[1:], 1):
            acc.add_(_shifted(padded, halo, axis, -k), alpha=c).add_(_shifted(padded, halo, axis, k), alpha=c)
    return acc


def _padded(level, halo, periodic=False):
    if periodic:
        return torch.nn.functional.pad(level[None, None], (halo,) * (2 * level.dim()), mode="circular")[0, 0]
    return torch.nn.functional.pad(level, (halo,) * (2 * level.dim()))


def _corners(shape, pos):
    """Grid points and multilinear weights of positions off the grid (a grid point has one corner)."""
    found = []
    for p in pos:
        around = [((), 1.0)]
        for x, n in zip(p, shape):
            b = min(int(math.floor(x)), n - 2)
            around = [(at + (b + i,), w * f) for at, w in around for i, f in ((0, 1 - (x - b)), (1, x - b))]
        found.append(around)
    return found


def _exact_wave(case, x):
    shape, r, c = x["shape"], x["radius"], x["coeffs"]
    u, prev, beta = (x[k].double() for k in ("u", "prev", "beta"))
    if case["offgrid"]:
        src, rec = (_corners(shape, p if p is not None else ()) for p in (x["src"], x["rec"]))
    else:
        src, rec = ([[(tuple(int(i) for i in q), 1.0)] for q in (p if p is not None else ())] for p in (x["src"], x["rec"]))
    gamma = None
    if case["layer"]:
        gamma = torch.zeros(shape, dtype=torch.float64, device=DEVICE)
        for d, p in enumerate(_profiles(shape, case["layer"])):
            at = [1] * len(shape)
            at[d] = -1
            gamma += torch.from_numpy(p).to(DEVICE).reshape(at)
    amp = x["amp"].cpu().numpy()
    trace = []
    for t in range(case["steps"]):
        new = _star(_padded(u, r, case["periodic"]), r, c).mul_(beta).add_(u, alpha=2.0)
        if gamma is None:
            new.sub_(prev)
        else:
            new.sub_((1.0 - gamma) * prev).div_(1.0 + gamma)
        for s, around in enumerate(src):
            for at, w in around:
                new[at] += w * amp[t, s]
        prev, u = u, new
        if rec:
            trace.append(sum(u[tuple(torch.tensor([p[i][0][d] for p in rec], device=DEVICE) for d in range(u.dim()))]
                             * torch.tensor([p[i][1] for p in rec], dtype=torch.float64, device=DEVICE)
                             for i in range(len(rec[0]))))
    return u, prev, torch.stack(trace) if trace else None


def _exact_sweep(case, seed):
    x = _sweep_inputs(case, seed)
    if case["kind"] == "heat":
        u = x["u"].double()
        for _ in range(case["steps"]):
            u = u + _star(_padded(u, x["radius"], case["periodic"]), x["radius"], x["coeffs"])
        return {"u": u}
    u, prev, trace = _exact_wave(case, x)
    out = {} if trace is None else {"trace": trace}
    out["u"], out["prev"] = u, prev
    return out


def _exact_batch(case, seed):
    out = []
    for i, shape in enumerate(_shot_shapes(case, seed)):
        shot = _shot_case(case, shape)
        out.append(list(_exact_wave(shot, _sweep_inputs(shot, seed + 7919 * i))[:2]))
    return out


def _exact_gradient(case, seed):
    x = _gradient_inputs(case, seed)
    shape, m, dt, n = x["shape"], x["m"], x["dt"], case["steps"]
    c = S.second_derivative_weights(8)
    beta = dt * dt / (H * H * m)
    at = tuple(torch.from_numpy(x["rec"][:, d].copy()).to(DEVICE) for d in range(3))
    src = tuple(int(i) for i in x["src"][0])
    amount = x["wavelet"][:, 0] * (dt * dt / m[src])
    zero = torch.zeros(shape, dtype=torch.float64, device=DEVICE)
    u, prev, trace, second = zero, zero, [], []
    for t in range(n):
        new = _star(_padded(u, 4), 4, c) * beta + 2.0 * u - prev
        new[src] += amount[t]
        trace.append(new[at])
        second.append(new - 2.0 * u + prev)
        prev, u = u, new
    trace = torch.stack(trace)
    resid = trace - x["d_obs"]
    weight = dt * dt / m[at]
    lam, after, grad = zero, zero, torch.zeros_like(zero)
    for t in range(n - 1, -1, -1):
        new = _star(_padded(lam, 4), 4, c) * beta + 2.0 * lam - after
        new.index_put_(at, weight * resid[t], accumulate=True)
        after, lam = lam, new
        grad -= lam * second[t] / (dt * dt)
    return {"misfit": 0.5 * resid.square().sum().reshape(1), "grad": grad, "trace": trace}


def _exact_program(case, seed):
    v = [p.double() for p in _velocities(_shape(case), seed)]

    def at(field, off):
        return v[field][tuple(slice(1 + o, n - 1 + o) for o, n in zip(off, v[field].shape))]

    out = [torch.zeros(_shape(case), dtype=torch.float64, device=DEVICE) for _ in range(3)]
    for o, coeff, factors in pw_advection_terms(1.0, 1.0, 1.0):
        out[o] += coeff * math.prod(at(f, off) for f, off in factors)
    return out


def _exact_rank(case, seed):
    x = _sweep_inputs(_sweep("", "wave", _shape(case), 8, case["steps"], dtype=case["dtype"]), seed)
    u, prev, beta = (x[k].double() for k in ("u", "prev", "beta"))
    for _ in range(case["steps"]):
        p = _padded(u, 4)
        p[:4, 4:-4, 4:-4], p[-4:, 4:-4, 4:-4] = u[:4], u[-4:]
        u, prev = _star(p, 4, x["coeffs"]) * beta + 2.0 * u - prev, u
    return {"u": u, "prev": prev}
