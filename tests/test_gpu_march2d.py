"""The 2D sweep by strips: one step per launch against the one-thread-per-point
apply, and passes of several steps against single steps, bit for bit; at
ragged sizes, with sources and receivers at the edges of strips and chunks,
with halos that are not zero, and with more sources in a row than a pass takes."""
import numpy as np
import pytest

import paper_2404_02218_amd as S

pytestmark = pytest.mark.gpu


def _weights(kind, radius):
    return S.heat_weights(2 * radius, 0.05) if kind == S.HEAT else S.second_derivative_weights(2 * radius)


def _fields(plan, seed, halo_values=False):
    """Random levels (and beta); halos zero, or random with NaN corners, which no star reads."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    r, f = plan.halo, [plan.field() for _ in range(3 if plan.kind == S.WAVE2 else 2)]
    for x in f[:2]:
        if halo_values:
            x.view.copy_(torch.randn(x.view.shape, generator=g, device="cuda"))
            for a in (slice(0, r), slice(-r, None)):
                for b in (slice(0, r), slice(-r, None)):
                    x.view[a, b] = float("nan")
        else:
            x.view[r:-r, r:-r] = torch.randn(plan.shape, generator=g, device="cuda").to(x.view.dtype)
    if len(f) > 2:
        f[2].view.copy_(torch.rand(f[2].view.shape, generator=g, device="cuda") * 0.05)
    return f


def _bits(f):
    import torch
    return f.view.contiguous().view(torch.int32 if f.dtype == S.F32 else torch.int16)


@pytest.mark.parametrize("shape", [(1, 1), (3, 5), (16, 240), (17, 241), (4, 224), (5, 225), (33, 700)])
@pytest.mark.parametrize("radius,dtype", [(1, S.F32), (2, S.BF16), (3, S.F16), (4, S.F32)])
@pytest.mark.parametrize("kind", [S.HEAT, S.WAVE2])
def test_step_equals_apply(device, kind, radius, dtype, shape):
    import torch
    plan = S.Plan(kind, shape, radius, _weights(kind, radius), dtype=dtype)
    plan.variant = 0
    f = _fields(plan, 1, halo_values=True)
    for _ in range(3):
        want = plan.field()
        want.storage.copy_(f[1].storage)
        plan.apply(want, f)
        plan.run(f, 1)
        assert torch.equal(_bits(f[0]), _bits(want))


def _points(shape, radius, n, rng):
    """Points at the corners, at strip ends and chunk rows, two of them coincident."""
    width = 256 - 2 * (-(-radius * (8 if radius == 1 else 4) // 4) * 4)
    ny, nx = shape
    p = [(0, 0), (ny - 1, nx - 1), (ny // 2, width - 1), (ny // 2, width), (7, 2 * width), (7, 2 * width)]
    p += [(int(rng.integers(ny)), int(rng.integers(nx))) for _ in range(n - len(p))]
    return np.array(p)


@pytest.mark.parametrize("kind,radius,dtype,shape", [
    (S.HEAT, 1, S.F32, (1103, 1201)), (S.HEAT, 1, S.F32, (2003, 2101)), (S.HEAT, 2, S.F32, (2503, 2402)),
    (S.HEAT, 1, S.F16, (2901, 2803)), (S.WAVE2, 1, S.F32, (997, 1001)), (S.WAVE2, 1, S.F32, (2003, 2101)),
    (S.WAVE2, 2, S.F32, (3001, 1003)), (S.WAVE2, 3, S.F32, (1999, 2601)), (S.WAVE2, 4, S.F32, (2999, 3013)),
    (S.WAVE2, 1, S.BF16, (2501, 2499)), (S.WAVE2, 2, S.F16, (3801, 3703))])
@pytest.mark.parametrize("halo_values", [False, True])
def test_passes_equal_single_steps(device, kind, radius, dtype, shape, halo_values):
    import torch
    n = 29   # passes of 8, then 4, then steps
    rng = np.random.default_rng(radius)
    src, rec = _points(shape, radius, 12, rng), _points(shape, radius, 90, rng)
    rec[20:] = np.stack([np.full(70, 9), rng.integers(0, shape[1], 70)], axis=1)
    amp = torch.from_numpy(rng.standard_normal((n, len(src)))).cuda()
    trace = torch.zeros((2, n, len(rec)), dtype=torch.float64, device=device)
    plan = S.Plan(kind, shape, radius, _weights(kind, radius), dtype=dtype)
    plan.variant = 0
    assert (plan.run_workspace_bytes() > 0) == (kind == S.WAVE2)   # large enough for passes
    a = _fields(plan, 2, halo_values)
    plan.run(a, n, src=src, src_amp=amp, rec=rec, rec_trace=trace[0])
    b = _fields(plan, 2, halo_values)
    for t in range(n):
        plan.run(b, 1, src=src, src_amp=amp[t:t + 1], rec=rec, rec_trace=trace[1, t:t + 1])
    assert torch.equal(_bits(a[0]), _bits(b[0]))
    if kind == S.WAVE2:
        assert torch.equal(_bits(a[1]), _bits(b[1]))
    assert torch.equal(trace[0], trace[1]) and float(trace[0].abs().max()) > 0


def test_a_wave_plan_without_a_workspace_steps(device):
    import ctypes as C
    import torch
    plan = S.Plan(S.WAVE2, (1000, 1003), 1, _weights(S.WAVE2, 1))
    a, b = _fields(plan, 3), _fields(plan, 3)
    ptrs = (C.c_void_p * 3)(*[f.ptr for f in a])
    S.call("stencil_run", plan.handle, ptrs, 16, None, None, None)   # none was attached
    plan.run(b, 16)
    assert torch.equal(_bits(a[0]), _bits(b[0])) and torch.equal(_bits(a[1]), _bits(b[1]))


@pytest.mark.parametrize("count", [16, 17, 150])
def test_many_sources_in_a_row(device, count):
    import torch
    plan = S.Plan(S.HEAT, (1100, 1111), 1, _weights(S.HEAT, 1))
    plan.variant = 0
    src = np.stack([np.full(count, 501), 300 + np.arange(count) // 2], axis=1)
    amp = torch.randn((16, count), dtype=torch.float64, device=device)
    a, b = _fields(plan, 4), _fields(plan, 4)
    plan.run(a, 16, src=src, src_amp=amp)
    for t in range(16):
        plan.run(b, 1, src=src, src_amp=amp[t:t + 1])
    assert torch.equal(_bits(a[0]), _bits(b[0]))


@pytest.mark.parametrize("radius,shape", [(1, (1001, 1003)), (4, (2999, 3013))])
def test_damped_passes_equal_single_steps(device, radius, shape):
    import torch
    plan = S.Plan(S.WAVE2, shape, radius, _weights(S.WAVE2, radius))
    plan.set_damping([S.damping_profile(k, 20, 0.1) for k in shape])
    a, b = _fields(plan, 5), _fields(plan, 5)
    plan.run(a, 16)
    for _ in range(16):
        plan.run(b, 1)
    assert torch.equal(_bits(a[0]), _bits(b[0])) and torch.equal(_bits(a[1]), _bits(b[1]))


@pytest.mark.parametrize("radius,shape", [(1, (50, 77)), (1, (100, 3)), (2, (33, 130)), (2, (70, 45))])
@pytest.mark.parametrize("halo_values", [False, True])
def test_multistep_heat_keeps_the_halo(device, radius, shape, halo_values):
    """The multi-step tiles against the sweep by strips, with any halo and any number of steps."""
    import torch
    plan = S.Plan(S.HEAT, shape, radius, _weights(S.HEAT, radius))
    for nsteps in (1, 2, 7, 15, 40):
        plan.variant = 0
        want = _fields(plan, 6, halo_values)
        plan.run(want, nsteps)
        for v in range(1, plan.variant_count()):
            plan.variant = v
            f = _fields(plan, 6, halo_values)
            plan.run(f, nsteps)
            r = plan.halo
            assert torch.equal(f[0].view[r:-r, r:-r], want[0].view[r:-r, r:-r]), (plan.variant_name(v), nsteps)


@pytest.mark.parametrize("shape", [(3, 200), (40, 700)])
@pytest.mark.parametrize("kind", [S.HEAT, S.WAVE2])
def test_step_with_more_points_than_lanes(device, kind, shape):
    """150 sources and receivers, most of them in one strip, some coincident: each
    sweep adds them in the list's order and records the level that it wrote."""
    import torch
    rng = np.random.default_rng(9)
    plan = S.Plan(kind, shape, 2, _weights(kind, 2))
    plan.variant = 0
    src, rec = (np.stack([rng.integers(0, shape[0], 150), rng.integers(0, 200, 150)], axis=1) for _ in range(2))
    src[120:] = src[:30]
    amp = rng.standard_normal((1, 150))
    f = _fields(plan, 2)
    want = plan.field()
    want.storage.copy_(f[1].storage)
    plan.apply(want, f)
    level = want.view[2:-2, 2:-2].cpu().numpy()
    for (y, x), a in zip(src, amp[0]):
        level[y, x] = np.float32(np.float64(level[y, x]) + a)
    trace = torch.zeros((2, 150), dtype=torch.float64, device="cuda")
    amps = torch.tensor(np.concatenate([amp, np.zeros((1, 150))]), dtype=torch.float64, device="cuda")
    g = [plan.field() for _ in f]
    for a, b in zip(g, f):
        a.storage.copy_(b.storage)
    plan.run(f, 1, src=src, src_amp=amps[:1], rec=rec, rec_trace=trace[:1])
    assert np.array_equal(f[0].view[2:-2, 2:-2].cpu().numpy(), level)
    # row t of the trace is the level that step t wrote
    plan.run(g, 2, src=src, src_amp=amps, rec=rec, rec_trace=trace)
    rows = [a[rec[:, 0], rec[:, 1]].astype(np.float64) for a in (level, g[0].view[2:-2, 2:-2].cpu().numpy())]
    assert np.array_equal(trace.cpu().numpy(), rows)
