"""The brick kernel (variant 0 of 3D plans, and 3D applies on boxes) at the
edges of its bricks: it must give the z-marching sweep's bits, and touch
nothing outside a box."""
import numpy as np
import pytest

import paper_2404_02218_amd as S
import workloads as W
from _helpers import gpu_wave, torch_f64, wave_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [S.F32, S.BF16, S.F16])
@pytest.mark.parametrize("shape", [(1, 15, 63), (2, 16, 64), (5, 17, 65), (9, 33, 130)])
def test_many_sources_equal_zmarch(device, shape, dtype):
    # 150 sources, most in one plane of one brick, two of them coincident
    rng = np.random.default_rng(sum(shape))
    src = np.stack([rng.integers(0, n, 150) for n in shape], axis=1)
    src[:120, 0] = shape[0] - 1
    src[7] = src[3]
    amp = rng.standard_normal((5, 150))
    rec = np.stack([rng.integers(0, n, 20) for n in shape], axis=1)
    u0, um1, beta = wave_inputs(shape, seed=7, dtype=dtype)
    plan = S.Plan(S.WAVE2, shape, 4, S.second_derivative_weights(8), dtype=dtype)
    a = gpu_wave(plan, u0, um1, beta, 5, src=src, amp=amp, rec=rec, variant=0)
    b = gpu_wave(plan, u0, um1, beta, 5, src=src, amp=amp, rec=rec, variant=1)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("radius,dtype", [(1, S.F16), (3, S.F32), (4, S.F32), (4, S.BF16)])
@pytest.mark.parametrize("box", [((0, 0, 0), (9, 37, 141)), ((3, 5, 7), (4, 6, 8)), ((1, 16, 61), (9, 33, 66)),
                                 ((0, 2, 66), (5, 37, 135)), ((4, 4, 4), (4, 8, 8))])
def test_apply_on_a_box_equals_a_sweep(device, box, radius, dtype):
    import torch
    shape = (9, 37, 141)
    u0, um1, beta = wave_inputs(shape, seed=11, dtype=dtype, halo=radius)
    plan = S.Plan(S.WAVE2, shape, radius, S.second_derivative_weights(2 * radius), dtype=dtype)
    f = [plan.field().load(W.embed(a, radius)) for a in (u0, um1, beta)]
    want, _, _ = gpu_wave(plan, u0, um1, beta, 1, variant=1)
    lo, hi = box
    inside = tuple(slice(a, b) for a, b in zip(lo, hi))
    # in place over the previous level, and into another field
    other = plan.field().load(np.full(tuple(n + 2 * radius for n in shape), 3.0))
    for out in (other, f[1]):
        before = out.storage.clone()
        plan.apply(out, f, lo, hi)
        got = out.interior(radius)
        assert np.array_equal(got[inside], want[inside])
        view = before.as_strided(plan.layout.extents, plan.layout.strides, plan.layout.offset)
        sl = tuple(slice(radius + a, radius + b) for a, b in zip(lo, hi))
        view[sl] = out.view[sl]
        assert torch.equal(before.view(torch.uint8), out.storage.view(torch.uint8))


@pytest.mark.parametrize("shape", [(13, 21, 70), (20, 47, 64)])
def test_gradient_equals_zmarch(device, shape):
    import torch
    rng = np.random.default_rng(5)
    n, every = 11, 4
    v = rng.uniform(1500, 4500, shape)
    m = torch_f64(1.0 / v ** 2, device)
    dt = W.wave_dt(4500.0, 10.0)
    wavelet = torch_f64(W.ricker(np.arange(n) * dt, 60.0).reshape(-1, 1), device)
    d_obs = torch_f64(rng.standard_normal((n, 80)), device)
    rec = np.stack([np.full(80, 5), rng.integers(0, shape[1], 80), rng.integers(0, shape[2], 80)], axis=1)
    got = []
    for variant in (0, 1, 2):
        plan = S.Plan(S.WAVE2, shape, 4, S.second_derivative_weights(8))
        plan.variant = variant
        f = [plan.field() for _ in range(3)]
        ws = torch.empty(plan.adjoint_workspace_bytes(n, every), dtype=torch.uint8, device=device)
        trace = torch.zeros((n, 80), dtype=torch.float64, device=device)
        J = torch.zeros(1, dtype=torch.float64, device=device)
        grad = torch.zeros(shape, dtype=torch.float64, device=device)
        plan.gradient(f, m, dt, 10.0, n, every, ws, [[5, 9, 20]], wavelet, rec, trace, d_obs, J, grad)
        got.append((trace, J, grad))
    assert float(got[0][2].abs().max()) > 0
    for g in got[1:]:
        for x, y in zip(got[0], g):
            assert torch.equal(x, y)


def test_heat_sources_are_added_after_the_step(device):
    shape = (6, 20, 70)
    u0 = W.round_to_storage(np.random.default_rng(3).random(shape), "f32")
    plan = S.Plan(S.HEAT, shape, 2, S.heat_weights(4, 0.05))
    plan.variant = 0
    out = []
    for src in (None, [[5, 19, 69], [0, 3, 64], [5, 19, 69]]):
        f = [plan.field().load(W.embed(u0, 2)), plan.field()]
        amp = torch_f64([[0.5, -0.25, 0.125]], device) if src else None
        plan.run(f, 1, src=src, src_amp=amp)
        out.append(f[0].interior(2))
    want = out[0].astype(np.float32)
    for at, a in (((5, 19, 69), 0.5), ((0, 3, 64), -0.25), ((5, 19, 69), 0.125)):
        want[at] = np.float32(np.float64(want[at]) + a)
    assert np.array_equal(out[1], want.astype(np.float64))


@pytest.mark.parametrize("dtype,sides,nsteps", [(S.F32, [(17, 40, 70), (9, 16, 64), (40, 37, 65)], 5),
                                               (S.BF16, [(17, 40, 70), (9, 16, 64)], 4),
                                               (S.F32, [(190, 190, 190), (24, 24, 24), (180, 190, 200), (186, 186, 186)], 7)])
def test_batch_in_bricks_equals_single_runs(device, dtype, sides, nsteps):
    """Several shots per launch, and (the large ones) several groups of shots."""
    import torch
    batch = S.BatchPlan(sides, 4, S.second_derivative_weights(8), dtype=dtype)
    batch.variant = 19
    assert batch.variant_name(19) == "zmarch_64x16_t256_zc32"
    g = torch.Generator(device="cuda").manual_seed(3)
    rng = np.random.default_rng(3)
    start, want, srcs, amps, recs = [], [], [], [], []
    for i, shape in enumerate(sides):
        f = [batch.field(i) for _ in range(3)]
        for x in f[:2]:
            x.view[4:-4, 4:-4, 4:-4] = torch.randn(shape, generator=g, device="cuda").to(x.view.dtype)
        f[2].view.uniform_(0.005, 0.05, generator=g)
        srcs.append(np.stack([rng.integers(0, n, 3) for n in shape], axis=1))
        recs.append(np.stack([rng.integers(0, n, 5) for n in shape], axis=1))
        amps.append(torch.from_numpy(rng.standard_normal((nsteps, 3))).cuda())
        start.append(f)
        plan = S.Plan(S.WAVE2, shape, 4, S.second_derivative_weights(8), dtype=dtype)
        plan.variant = 1
        h = [plan.field() for _ in range(3)]
        for a, b in zip(h, f):
            a.storage.copy_(b.storage)
        trace = torch.zeros((nsteps, 5), dtype=torch.float64, device=device)
        plan.run(h, nsteps, src=srcs[i], src_amp=amps[i], rec=recs[i], rec_trace=trace)
        want.append((h[0].storage, h[1].storage, trace))
    traces = [torch.zeros((nsteps, 5), dtype=torch.float64, device=device) for _ in sides]
    batch.run(start, nsteps, srcs=srcs, src_amps=amps, recs=recs, rec_traces=traces)
    for f, t, w in zip(start, traces, want):
        assert torch.equal(f[0].storage, w[0]) and torch.equal(f[1].storage, w[1]) and torch.equal(t, w[2])
