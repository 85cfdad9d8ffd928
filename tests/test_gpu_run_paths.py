"""Runs that change their route between calls (an attached workspace that
shrinks, a capture of the caller's), against plain runs."""
import ctypes as C

import numpy as np
import pytest

import paper_2404_02218_amd as S

pytestmark = pytest.mark.gpu


def _weights(kind, radius):
    return S.heat_weights(2 * radius, 0.05) if kind == S.HEAT else S.second_derivative_weights(2 * radius)


def _fields(plan, seed):
    """Random levels (and beta), zero halos."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    h, f = plan.halo, [plan.field() for _ in range(3 if plan.kind == S.WAVE2 else 2)]
    inner = (slice(h, -h),) * plan.ndim
    for x in f[:2]:
        x.view[inner] = torch.randn(plan.shape, generator=g, device="cuda").to(x.view.dtype)
    if len(f) > 2:
        f[2].view.copy_(torch.rand(f[2].view.shape, generator=g, device="cuda") * 0.05)
    return f


def _bits(f):
    import torch
    return f.view.contiguous().view(torch.int32 if f.dtype == S.F32 else torch.int16)


def _same(a, b):
    import torch
    return all(torch.equal(_bits(x), _bits(y)) for x, y in zip(a, b))


def _run(plan, f, nsteps):
    """stencil_run itself, with the workspace that is attached."""
    ptrs = (C.c_void_p * 3)(*[x.ptr for x in f] + [0] * (3 - len(f)))
    S.call("stencil_run", plan.handle, ptrs, nsteps, None, None, None)
    if ptrs[0] != f[0].ptr:
        f[0], f[1] = f[1], f[0]


def test_a_shrunk_workspace_is_not_written_past_its_end(device):
    import torch
    plan = S.Plan(S.WAVE2, (1300, 1303), 1, _weights(S.WAVE2, 1))
    need = plan.run_workspace_bytes()
    assert need > 0
    buf = torch.full((need,), 0x5a, dtype=torch.uint8, device=device)
    f, want = _fields(plan, 3), _fields(plan, 3)
    for nbytes in (need, need // 2, need, 4096):
        S.call("stencil_set_workspace", plan.handle, C.c_void_p(buf.data_ptr()), nbytes, None)
        buf[nbytes:] = 0x5a
        for _ in range(3):
            _run(plan, f, 16)
        S.call("stencil_set_workspace", plan.handle, None, 0, None)
        for _ in range(48):
            _run(plan, want, 1)
        assert torch.all(buf[nbytes:] == 0x5a)
        assert _same(f, want)


@pytest.mark.parametrize("kind,shape", [(S.WAVE2, (40, 44, 72)), (S.WAVE2, (162, 162, 162)), (S.HEAT, (70, 90)),
                                        (S.WAVE2, (2100, 2050))])
@pytest.mark.parametrize("kept", [1, 3])
def test_runs_in_a_caller_capture(device, kind, shape, kept):
    """Runs captured by the caller, before and after the plan has a graph of its own, replayed three times with
    eager work between."""
    import torch
    n, rng = 6, np.random.default_rng(5)
    src = np.stack([rng.integers(0, k, 3) for k in shape], axis=1)
    rec = np.stack([rng.integers(0, k, 9) for k in shape], axis=1)
    amp = torch.from_numpy(rng.standard_normal((n, 3))).cuda()
    plan = S.Plan(kind, shape, 2, _weights(kind, 2))
    plan.variant = 0
    points = dict(src=src, src_amp=amp, rec=rec)

    def passes(f, trace, captured):
        inner = (slice(2, -2),) * len(shape)
        out, graph = [], None
        for _ in range(kept):
            plan.run(f, n, rec_trace=trace, **points)
        if captured:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                plan.run(f, n, rec_trace=trace, **points)
                plan.run(f, n, rec_trace=trace, **points)
        for k in range(3):
            f[0].view[inner] *= 0.5 + 0.1 * k
            if captured:
                graph.replay()
            else:
                plan.run(f, n, rec_trace=trace, **points)
                plan.run(f, n, rec_trace=trace, **points)
            torch.cuda.synchronize()
            out.append([x.view.clone() for x in f] + [trace.clone()])
        return out

    trace = torch.zeros((n, 9), dtype=torch.float64, device=device)
    got = passes(_fields(plan, 7), trace, True)
    want = passes(_fields(plan, 7), trace, False)
    for a, b in zip(got, want):
        assert all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("shape,radius", [((70, 90), 1), ((130, 75), 2), ((1400, 1203), 1), ((20, 40, 70), 2)])
@pytest.mark.parametrize("noalloc", [False, True])
def test_heat_points_are_served_by_every_variant(device, shape, radius, noalloc):
    """Sources and receivers of a heat run at every variant and the default one, against single steps."""
    import torch
    n, rng = 9, np.random.default_rng(4)
    src = np.stack([rng.integers(0, k, 5) for k in shape], axis=1)
    src[4] = src[2]
    rec = np.stack([rng.integers(0, k, 80) for k in shape], axis=1)
    rec[:5] = src
    amp = torch.from_numpy(rng.standard_normal((n, 5))).cuda()
    plan = S.Plan(S.HEAT, shape, radius, _weights(S.HEAT, radius))
    default = plan.variant

    def run(f, t0, n):
        trace = torch.zeros((n, 80), dtype=torch.float64, device=device)
        sp, rp = S._Points(src, amp[t0:t0 + n].contiguous()), S._Points(rec, trace)
        ptrs = (C.c_void_p * 3)(*[x.ptr for x in f] + [0])
        S.call("stencil_run_noalloc" if noalloc else "stencil_run", plan.handle, ptrs, n, C.byref(sp.source()),
               C.byref(rp.receivers()), None)
        torch.cuda.synchronize()
        if ptrs[0] != f[0].ptr:
            f[0], f[1] = f[1], f[0]
        return trace

    plan.variant = 0
    want = _fields(plan, 2)
    rows = torch.cat([run(want, t, 1) for t in range(n)])
    for v in [default] + list(range(plan.variant_count())):
        plan.variant = v
        f = _fields(plan, 2)
        assert torch.equal(run(f, 0, n), rows), plan.variant_name(v)
        assert _same(f[:1], want[:1]), plan.variant_name(v)


def test_a_large_2d_wave_runs_where_its_workspace_does_not_fit(device, monkeypatch):
    import torch
    plan, other = (S.Plan(S.WAVE2, (1300, 1303), 1, _weights(S.WAVE2, 1)) for _ in range(2))
    f, want = _fields(plan, 3), _fields(plan, 3)
    real = torch.empty

    def empty(*size, **kw):
        if size == (plan.run_workspace_bytes(),):
            raise torch.cuda.OutOfMemoryError("out of memory")
        return real(*size, **kw)

    monkeypatch.setattr(torch, "empty", empty)
    for _ in range(3):
        plan.run(f, 16)
    monkeypatch.undo()
    for _ in range(3):
        other.run(want, 16)
    assert plan._ws.buf is None and other._ws.buf is not None
    assert _same(f, want)


@pytest.mark.parametrize("kind,shape,radius,dtype", [(S.WAVE2, (1300, 1303), 1, S.F32), (S.WAVE2, (700, 803), 4, S.F16),
                                                     (S.HEAT, (1300, 1111), 1, S.F32), (S.WAVE2, (64, 80, 150), 4, S.F32),
                                                     (S.HEAT, (64, 80, 150), 1, S.BF16)])
@pytest.mark.parametrize("nsrc,nrec", [(10, 90), (40, 0), (300000, 70), (3, 400000)])
def test_noalloc_equals_run_by_strips_and_bricks(device, kind, shape, radius, dtype, nsrc, nrec):
    """Lists that the scratch array holds by strip or tile, with coincident sources and more than 16 in a row, and
    lists (past 260,000 points) that it holds by position only."""
    import torch
    n, rng = 17, np.random.default_rng(6)
    src = np.stack([rng.integers(0, k, nsrc) for k in shape], axis=1)
    if nsrc == 40:
        src[:, :-1], src[:, -1] = src[0, :-1], 300 % shape[-1] + np.arange(40) // 2
    src[-1] = src[0]
    rec = np.stack([rng.integers(0, k, nrec) for k in shape], axis=1) if nrec else None
    amp = torch.from_numpy(rng.standard_normal((n, nsrc))).cuda()
    plan = S.Plan(kind, shape, radius, _weights(kind, radius), dtype=dtype)
    plan.variant = 0
    plan._ws.ensure(plan.handle)
    out = []
    for name in ("stencil_run", "stencil_run_noalloc"):
        f = _fields(plan, 8)
        trace = torch.zeros((n, max(nrec, 1)), dtype=torch.float64, device=device)
        sp, rp = S._Points(src, amp), S._Points(rec, trace)
        r = rp.receivers()
        ptrs = (C.c_void_p * 3)(*[x.ptr for x in f] + [0] * (3 - len(f)))
        S.call(name, plan.handle, ptrs, n, C.byref(sp.source()), C.byref(r) if r else None, None)
        torch.cuda.synchronize()
        out.append((f, trace))
    assert _same(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert nrec == 0 or float(out[0][1].abs().max()) > 0


def _ab(plan, n, a, b, **points):
    """The fields and the trace of a run at variant a (or of single steps for None) and at variant b."""
    import torch
    out = []
    for v in (a, b):
        plan.variant = 0 if v is None else v
        f = _fields(plan, 9)
        rec, amp = points.get("rec"), points.get("src_amp")
        trace = torch.zeros((n, len(rec)), dtype=torch.float64, device="cuda") if rec is not None else None
        for t0, k in [(t, 1) for t in range(n)] if v is None else [(0, n)]:
            plan.run(f, k, src=points.get("src"), src_amp=amp[t0:t0 + k].contiguous() if amp is not None else None,
                     rec=rec, rec_trace=trace[t0:t0 + k] if trace is not None else None)
        out.append((f, trace))
    return out


@pytest.mark.parametrize("shape,dtype", [((9, 33, 130), S.F32), ((21, 16, 64), S.F32), ((40, 50, 70), S.BF16),
                                         ((6, 531, 1101), S.F16)])
@pytest.mark.parametrize("count", [64, 65, 700, 6000])
def test_long_lists_in_bricks_equal_zmarch(device, shape, dtype, count):
    """Lists past the 64 entries that a brick reads at once: spread, in one plane, in one column of bricks, with
    coincident points; and as many receivers as several recording workgroups take."""
    import torch
    n, rng = 4, np.random.default_rng(count)
    plan = S.Plan(S.WAVE2, shape, 4, _weights(S.WAVE2, 4), dtype=dtype)
    spread = np.stack([rng.integers(0, k, count) for k in shape], axis=1)
    plane, column = spread.copy(), spread.copy()
    plane[:, 0] = shape[0] - 2
    column[:, 1:] = np.minimum(column[:, 1:], 15)
    amp = torch.from_numpy(rng.standard_normal((n, count))).cuda()
    for src in (spread, plane, column):
        src[count // 2] = src[0]
        (f, tf), (g, tg) = _ab(plan, n, 0, 1, src=src, src_amp=amp, rec=spread)
        assert _same(f, g) and torch.equal(tf, tg)


def test_long_lists_in_the_gradient_equal_zmarch(device):
    """A full surface of receivers, whose residuals are the adjoint's sources: 1024 in one plane of a brick."""
    import torch
    shape, n, every = (20, 37, 150), 7, 3
    rng = np.random.default_rng(2)
    surface = np.stack([a.ravel() for a in np.meshgrid([5], range(37), range(150), indexing="ij")], axis=1)
    m = torch.from_numpy(1.0 / rng.uniform(1500, 4500, shape) ** 2).cuda()
    wavelet = torch.from_numpy(rng.standard_normal((n, 1))).cuda()
    d_obs = torch.from_numpy(rng.standard_normal((n, len(surface)))).cuda()
    got = []
    for variant in (0, 1):
        plan = S.Plan(S.WAVE2, shape, 4, _weights(S.WAVE2, 4))
        plan.variant = variant
        f = [plan.field() for _ in range(3)]
        ws = torch.empty(plan.adjoint_workspace_bytes(n, every), dtype=torch.uint8, device=device)
        trace, misfit = torch.zeros_like(d_obs), torch.zeros(1, dtype=torch.float64, device=device)
        grad = torch.zeros(shape, dtype=torch.float64, device=device)
        plan.gradient(f, m, 1e-3, 10.0, n, every, ws, [[5, 9, 20]], wavelet, surface, trace, d_obs, misfit, grad)
        got.append((trace, misfit, grad))
    assert float(got[0][2].abs().max()) > 0
    assert all(torch.equal(x, y) for x, y in zip(*got))


@pytest.mark.parametrize("kind,shape,radius,dtype", [(S.WAVE2, (70, 500), 4, S.F32), (S.HEAT, (64, 1000), 1, S.F16),
                                                     (S.WAVE2, (1300, 1303), 1, S.F32), (S.HEAT, (1200, 1001), 1, S.F32)])
@pytest.mark.parametrize("nsrc,nrec", [(65, 64), (3000, 0), (12, 5000), (1, 70000)])
def test_long_lists_in_strips_equal_single_entries(device, kind, shape, radius, dtype, nsrc, nrec):
    """Long lists of a strip, in passes of several steps and in single steps, against points applied to the fields
    after steps without them."""
    import torch
    n, rng = 17, np.random.default_rng(nsrc)
    at = rng.choice(shape[0] * shape[1], size=nsrc, replace=False)
    src = np.stack([at // shape[1], at % shape[1]], axis=1)
    amp = torch.from_numpy(rng.standard_normal((n, nsrc))).cuda()
    rec = np.stack([rng.integers(0, k, nrec) for k in shape], axis=1) if nrec else None
    plan = S.Plan(kind, shape, radius, _weights(kind, radius), dtype=dtype)
    (f, tf), (g, tg) = _ab(plan, n, None, 0, src=src, src_amp=amp, rec=rec)
    assert _same(f, g) and (rec is None or torch.equal(tf, tg))
    # the points applied to the fields after each step without them
    h, want = _fields(plan, 9), []
    inner = (slice(plan.halo, -plan.halo),) * 2
    for t in range(3):
        plan.run(h, 1)
        level = h[0].view[inner]
        y, x = (torch.from_numpy(src[:, d]).cuda() for d in range(2))
        level[y, x] = (level[y, x].double() + amp[t]).to(level.dtype)
        if rec is not None:
            want.append(level[torch.from_numpy(rec[:, 0]).cuda(), torch.from_numpy(rec[:, 1]).cuda()].double())
    k = _fields(plan, 9)
    trace = torch.zeros((3, max(nrec, 1)), dtype=torch.float64, device=device)
    plan.run(k, 3, src=src, src_amp=amp[:3].contiguous(), rec=rec, rec_trace=trace if nrec else None)
    assert _same(h[:1], k[:1])
    assert rec is None or torch.equal(torch.stack(want), trace)


@pytest.mark.parametrize("shape,rec,bound", [((1000, 1000), "all", 100.0), ((48, 400, 500), "surface", 150.0)])
def test_long_receiver_lists_are_not_walked_by_every_wave(device, shape, rec, bound):
    """us a step, from the difference of 40 and 240 steps a call.  One thread per receiver takes 12 and 71 with the
    sweep; every wave walking its strip's list took 940, one workgroup for all receivers 370."""
    import time

    import torch
    at = [range(k) for k in shape] if rec == "all" else [[6], range(shape[1]), range(shape[2])]
    at = np.stack([a.ravel() for a in np.meshgrid(*at, indexing="ij")], axis=1)
    plan = S.Plan(S.WAVE2, shape, 4, _weights(S.WAVE2, 4))
    plan.variant = 0
    f, best = _fields(plan, 1), []
    for n in (40, 240):
        trace = torch.zeros((n, len(at)), dtype=torch.float64, device=device)
        times = []
        for _ in range(4):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            plan.run(f, n, rec=at, rec_trace=trace)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        best.append(min(times))
    us = (best[1] - best[0]) / 200 * 1e6
    print(f"{us:.1f} us a step")
    assert us < bound


@pytest.mark.parametrize("dtype", [S.F32, S.BF16])
def test_a_batch_in_bricks_equals_the_zmarch(device, dtype):
    """Several groups of shots, with receivers and a list of more than 64 sources in a tile."""
    import torch
    sides, n, rng = [(190, 190, 190), (24, 24, 24), (180, 190, 200), (17, 40, 70), (186, 186, 186)], 5, np.random.default_rng(3)
    batch = S.BatchPlan(sides, 4, _weights(S.WAVE2, 4), dtype=dtype)
    names = {batch.variant_name(v): v for v in range(1, batch.variant_count())}
    srcs = [np.stack([rng.integers(0, k, 3 if i else 400) for k in s], axis=1) for i, s in enumerate(sides)]
    srcs[0][:, 1:] %= 16
    recs = [np.stack([rng.integers(0, k, 300) for k in s], axis=1) for s in sides]
    amps = [torch.from_numpy(rng.standard_normal((n, len(s)))).cuda() for s in srcs]
    got = []
    for name in ("bricks_64x16x2_t256", "zmarch_64x16_t256_zc32"):
        batch.variant = names[name]
        g = torch.Generator(device="cuda").manual_seed(3)
        f = [[batch.field(i) for _ in range(3)] for i in range(len(sides))]
        for i, shot in enumerate(f):
            for x in shot[:2]:
                x.view[4:-4, 4:-4, 4:-4] = torch.randn(sides[i], generator=g, device="cuda").to(x.view.dtype)
            shot[2].view.copy_(torch.rand(shot[2].view.shape, generator=g, device="cuda") * 0.05)
        traces = [torch.zeros((n, 300), dtype=torch.float64, device=device) for _ in sides]
        batch.run(f, n, srcs=srcs, src_amps=amps, recs=recs, rec_traces=traces)
        got.append((f, traces))
    for a, b, s, t in zip(got[0][0], got[1][0], got[0][1], got[1][1]):
        assert _same(a, b) and torch.equal(s, t)


def _halo_fields(plan, seed):
    """Random levels and coefficients everywhere, the halo included: only the radius next to the interior is read."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    f = [plan.field() for _ in range(3 if plan.kind == S.WAVE2 else 2)]
    for x in f[:2]:
        x.view.copy_(torch.randn(x.view.shape, generator=g, device="cuda"))
        outer = plan.halo - plan.radius
        for d in range(plan.ndim if outer else 0):
            x.view.narrow(d, 0, outer).fill_(float("nan"))
            x.view.narrow(d, x.view.shape[d] - outer, outer).fill_(float("nan"))
    if len(f) > 2:
        f[2].view.copy_(torch.rand(f[2].view.shape, generator=g, device="cuda") * 0.05)
    return f


@pytest.mark.parametrize("kind,radius,dtype,shape,extra", [
    (S.WAVE2, 1, S.F32, (1303, 1301), 0), (S.WAVE2, 2, S.F32, (2003, 2101), 3), (S.WAVE2, 3, S.F32, (2703, 2501), 0),
    (S.WAVE2, 4, S.F32, (4603, 4601), 2), (S.WAVE2, 2, S.F16, (4203, 4203), 0), (S.HEAT, 2, S.F32, (2803, 2802), 2),
    (S.HEAT, 1, S.BF16, (3003, 3001), 5), (S.HEAT, 1, S.F32, (3, 600001), 1), (S.WAVE2, 1, S.F32, (600001, 3), 1)])
def test_passes_on_large_grids_equal_single_steps(device, kind, radius, dtype, shape, extra):
    """Grids past the lines from which passes of several steps are taken, halos wider than the radius among them."""
    import torch
    n, rng = 13, np.random.default_rng(radius)
    src = np.stack([rng.integers(0, k, 12) for k in shape], axis=1)
    rec = np.stack([rng.integers(0, k, 200) for k in shape], axis=1)
    amp = torch.from_numpy(rng.standard_normal((n, 12))).cuda()
    trace = torch.zeros((2, n, 200), dtype=torch.float64, device=device)
    plan = S.Plan(kind, shape, radius, _weights(kind, radius), halo=radius + extra, dtype=dtype)
    plan.variant = 0
    a, b = _halo_fields(plan, 2), _halo_fields(plan, 2)
    plan.run(a, n, src=src, src_amp=amp, rec=rec, rec_trace=trace[0])
    for t in range(n):
        plan.run(b, 1, src=src, src_amp=amp[t:t + 1], rec=rec, rec_trace=trace[1, t:t + 1])
    levels = 1 if kind == S.HEAT else 3   # the other buffer of a heat run holds no set level
    assert _same(a[:levels], b[:levels]) and torch.equal(trace[0], trace[1])
    assert float(trace[0].abs().max()) > 0 and not torch.isnan(trace[0]).any()


@pytest.mark.parametrize("radius,dtype,shape,extra", [
    (4, S.F32, (9, 271, 270), 0), (4, S.F32, (9, 271, 270), 4), (4, S.F32, (9, 1931, 1953), 0), (2, S.F32, (23, 1001, 1003), 3),
    (4, S.F16, (9, 531, 1101), 0), (4, S.BF16, (9, 531, 1101), 2), (3, S.F16, (9, 531, 1101), 1), (1, S.BF16, (7, 33, 130), 9)])
@pytest.mark.parametrize("kind", [S.HEAT, S.WAVE2])
def test_every_form_of_bricks_equals_zmarch(device, kind, radius, dtype, shape, extra):
    """Bricks of two and of four planes, numbered x first and z first, halos wider than the radius among them; and
    the apply on boxes of such fields."""
    import torch
    plan = S.Plan(kind, shape, radius, _weights(kind, radius), halo=radius + extra, dtype=dtype)
    out = []
    for v in (0, 1):
        plan.variant = v
        f = _halo_fields(plan, 4)
        plan.run(f, 3)
        out.append(f)
    assert _same(*out)
    first = _halo_fields(plan, 4)
    plan.variant = 1
    want = _halo_fields(plan, 4)
    plan.run(want, 1)
    got = plan.field()
    got.storage.copy_(first[1].storage)
    cut = [(0, k // 2 + 1, k) for k in shape]
    for z in range(2):
        for y in range(2):
            for x in range(2):
                lo, hi = [c[i] for c, i in zip(cut, (z, y, x))], [c[i + 1] for c, i in zip(cut, (z, y, x))]
                plan.apply(got, first, lo, hi)
    assert _same([got], want[:1])


@pytest.mark.parametrize("shape,extra", [((9, 271, 270), 4), ((9, 1931, 1953), 0)])
def test_damped_bricks_equal_zmarch(device, shape, extra):
    out = []
    plan = S.Plan(S.WAVE2, shape, 4, _weights(S.WAVE2, 4), halo=4 + extra)
    plan.set_damping([S.damping_profile(k, 4, 0.1) for k in shape])
    for v in (0, 1):
        plan.variant = v
        f = _halo_fields(plan, 4)
        plan.run(f, 3)
        out.append(f)
    assert _same(*out)
