"""Checks of the library's host code on the stand-in HIP calls of
hip_stand_in.cpp, each run in a process of its own:

    python _host_runtime.py <stand-in .so> <check>

Fields are addresses only (no kernel runs).  The process must not load a real
HIP runtime first, so torch is kept out of it.
"""
import ctypes as C
import os
import struct
import sys
import types

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FIELD0 = 1 << 40   # addresses of pretended fields


class Host:
    def __init__(self, stand_in):
        self.hip = C.CDLL(stand_in, mode=C.RTLD_GLOBAL)
        self.hip.stand_in_name.restype = C.c_char_p
        self.hip.stand_in_arg0.restype = C.c_void_p
        sys.modules["torch"] = types.ModuleType("torch")
        sys.path.insert(0, ROOT)
        import paper_2404_02218_amd as S
        self.S, self.lib, self.next = S, S.lib(), FIELD0

    def take(self, nbytes):
        """An address range of its own, with a gap of the same size behind it."""
        at = self.next
        self.next += 2 * ((nbytes + 255) // 256 * 256) + 256
        return at

    def fields(self, plan, n):
        return [self.take(plan.layout.bytes) for _ in range(n)]

    def run(self, plan, fields, nsteps, src=None, rec=None, name="stencil_run", stream=None):
        ptrs = (C.c_void_p * 3)(*fields + [0] * (3 - len(fields)))
        st = getattr(self.lib, name)(plan.handle, ptrs, nsteps, C.byref(src) if src else None,
                                     C.byref(rec) if rec else None, stream)
        return st, [ptrs[i] for i in range(len(fields))]

    def launches(self):
        """(kernel name, grid, first bytes of the first argument) since the last call."""
        out = [(self.hip.stand_in_name(i).decode(), self.hip.stand_in_grid(i),
                C.string_at(self.hip.stand_in_arg0(i), 128)) for i in range(self.hip.stand_in_launches())]
        self.hip.stand_in_clear()
        return out

    def counts(self):
        c = (C.c_int * 9)()
        self.hip.stand_in_counts(c)
        return dict(zip(("captures", "instantiated", "replays", "syncs", "execs", "graphs", "events", "streams",
                         "blocks"), c))


def _outputs(launch):
    """The fields a launch of the 2D sweep writes: u, prev, beta, out, out1 lead its descriptor."""
    return [p for p in struct.unpack("8Q", launch[2][:64])[3:5] if p]


def shrunk_workspace(h):
    """A workspace attached again with fewer bytes, at the same address, is not written past them."""
    S = h.S
    plan = S.Plan(S.WAVE2, (4700, 4701), 4, S.second_derivative_weights(8))
    f, need = h.fields(plan, 3), plan.run_workspace_bytes()
    assert need > 0
    ws = h.take(need)
    for nbytes in (need, 4096, need, need // 2, 0, need):
        S.call("stencil_set_workspace", plan.handle, C.c_void_p(ws if nbytes else None), nbytes, None)
        h.launches()
        for _ in range(3):
            assert h.run(plan, f, 16)[0] == 0
            swept = [x for x in h.launches() if "2d" in x[0]]
            written = {p for x in swept for p in _outputs(x)} - set(f[:2])
            assert bool(written) == (nbytes == need) == any("k_march2d" in x[0] for x in swept)
            for p in written:
                assert ws <= p and p + plan.layout.bytes <= ws + nbytes


def _batch(h, sides, variant):
    S = h.S
    batch = S.BatchPlan(sides, 4, S.second_derivative_weights(8))
    batch.variant = next(v for v in range(batch.variant_count()) if batch.variant_name(v) == variant)
    return batch, [h.take(layout.bytes) for layout in batch.layouts for _ in range(3)]


def _run_batch(h, batch, fields, nsteps, stream=None):
    ptrs = (C.c_void_p * len(fields))(*fields)
    st = h.lib.stencil_batch_run(batch._h, ptrs, nsteps, None, None, stream)
    return st, list(ptrs)


def concurrent_batch(h):
    """Concurrent shots whose step count, buffers and variant change: one graph of four branches in the life
    of a plan, every launch in the run's own number and order of steps, and no handle left when it ends."""
    for sides in ([(20, 24, 28), (36, 40, 44), (17, 18, 19)], [(170, 170, 170), (60, 60, 60)]):   # past 2^22 points
        before = h.counts()
        batch, f = _batch(h, sides, "shots_concurrent_4")
        fused = next(v for v in range(batch.variant_count()) if batch.variant_name(v).startswith("zmarch_64x32"))
        concurrent = batch.variant
        for n in [7, 7, 38, 39, 40, 40, 40, 38, 39, 40, 2, 2, 2, 3, 4, 5, 6, 40, 40, 40]:
            h.launches()
            st, f = _run_batch(h, batch, f, n)
            assert st == 0
            assert sum("k_zbrick" in x[0] for x in h.launches()) == n * len(sides)
        for v in (fused, concurrent, fused, concurrent):
            batch.variant = v
            for _ in range(3):
                assert _run_batch(h, batch, f, 4)[0] == 0
        branched = h.counts()["captures"] - before["captures"]
        assert branched == 1 + 2   # and one of each run of the fused variant
        del batch
        after = h.counts()
        assert {k: after[k] for k in ("execs", "graphs", "events", "streams", "blocks")} == \
               {k: before[k] for k in ("execs", "graphs", "events", "streams", "blocks")}


def _delta(h, before):
    return {k: n - before[k] for k, n in h.counts().items()}


def runs_that_are_not_repeated(h):
    """Runs whose arguments change from call to call (an odd step count makes the fields change places) wait for
    nothing and cost no graph, but for one captured behind the first of them on a large grid; of a run that is
    repeated the third call replays at the latest."""
    S = h.S
    for shape in ((170, 170, 170), (40, 44, 48), (2100, 2050)):   # the first and last past 2^22 points
        plan = S.Plan(S.WAVE2, shape, 4, S.second_derivative_weights(8))
        plan.variant = 0
        f = h.fields(plan, 3)
        before = h.counts()
        for n in (5, 5, 7, 7, 7, 3, 4, 6, 4, 6):
            h.launches()
            st, f = h.run(plan, f, n)
            assert st == 0 and len(h.launches()) == n
        d = _delta(h, before)
        large = shape != (40, 44, 48)
        assert d["captures"] == large and d["syncs"] == 0, d
        want = None
        for k in range(5):   # direct, captured, replayed
            assert h.run(plan, f, 8)[0] == 0
            got = h.launches()
            assert len(got) == 8 and (want is None or got == want), shape
            want = got
        d = _delta(h, before)
        assert (d["captures"], d["execs"]) == (1 + large, 1) and d["replays"] >= 3
        # the next run is one again that may be repeated: captured behind the first call
        assert h.run(plan, f, 10)[0] == 0 and h.run(plan, f, 10)[0] == 0 and h.run(plan, f, 10)[0] == 0
        d = _delta(h, before)
        assert d["captures"] == 2 + large and d["replays"] >= 3 + 1 + large
        # a graph that was never launched is not waited for
        assert h.run(plan, f, 6)[0] == 0 and h.run(plan, f, 6)[0] == 0
        waited = h.counts()["syncs"]
        assert h.run(plan, f, 8)[0] == 0
        assert h.counts()["syncs"] - waited == (0 if _delta(h, before)["replays"] == d["replays"] else 1)
        del plan


def runs_in_a_caller_capture(h):
    """Runs on a stream that the caller is capturing are enqueued into that capture, whatever the plan has kept:
    nothing is waited for, no graph of the plan's is destroyed or launched there."""
    S = h.S
    stream = C.c_void_p()
    h.hip.hipStreamCreateWithFlags(C.byref(stream), 0)
    for shape in ((170, 170, 170), (40, 44, 48)):
        for kept in (1, 2, 3):   # runs before the capture (the first one uploads the plan's tables)
            plan = S.Plan(S.WAVE2, shape, 4, S.second_derivative_weights(8))
            plan.variant = 0
            f = h.fields(plan, 3)
            for _ in range(kept):
                assert h.run(plan, f, 4, stream=stream)[0] == 0
            h.launches()
            before = h.counts()
            assert h.hip.hipStreamBeginCapture(stream, 0) == 0
            for n in (4, 6, 4, 6, 6):
                assert h.run(plan, f, n, stream=stream)[0] == 0, h.lib.stencil_last_error()
            graph = C.c_void_p()
            assert h.hip.hipStreamEndCapture(stream, C.byref(graph)) == 0 and graph.value
            assert not h.launches()   # all of it went into the capture
            d = _delta(h, before)
            assert (d["captures"], d["execs"], d["replays"], d["syncs"]) == (1, 0, 0, 0), d
            x = C.c_void_p()
            assert h.hip.hipGraphInstantiate(C.byref(x), graph, None, None, C.c_size_t(0)) == 0
            assert h.hip.hipGraphLaunch(x, stream) == 0
            got = h.launches()
            assert len(got) == 26
            for n in (4, 6, 4, 6, 6):   # the same launches as outside
                assert h.run(plan, f, n)[0] == 0
            assert [g[2] for g in h.launches()] == [g[2] for g in got]
            h.hip.hipGraphExecDestroy(x)
            h.hip.hipGraphDestroy(graph)
            del plan


def _points(h, shape, n, step=1):
    """A list of n points of the grid, its positions kept alive with it."""
    pos = (C.c_int64 * (3 * n))()
    for k in range(n):
        at = k * step
        for d in range(len(shape) - 1, -1, -1):
            pos[3 * k + d] = at % shape[d]
            at //= shape[d]
    return pos


def heat_points(h):
    """A heat run with sources or receivers takes a sweep that serves them, whatever the variant; one without
    takes the multi-step sweep that the variant names.  So does the run without allocations."""
    S = h.S
    for shape, radius, multi in (((70, 90), 1, "k_heat2d_tb"), ((1300, 1301), 2, "k_heat2d_tb"), ((40, 44, 72), 2, "k_tb2")):
        plan = S.Plan(S.HEAT, shape, radius, S.heat_weights(2 * radius, 0.05))
        pos = _points(h, shape, 3, 1237)
        src = S.Source(3, C.cast(pos, C.c_void_p), C.c_void_p(4096), None)
        rec = S.Receivers(3, C.cast(pos, C.c_void_p), C.c_void_p(8192))
        f, seen = h.fields(plan, 2), 0
        for v in range(plan.variant_count()):
            plan.variant = v
            for name in ("stencil_run", "stencil_run_noalloc"):
                deep = []
                for points in ({}, {"src": src}, {"rec": rec}, {"src": src, "rec": rec}):
                    h.launches()
                    assert h.run(plan, f, 8, name=name, **points)[0] == 0
                    swept = [x[0] for x in h.launches() if "k_fill" not in x[0]]
                    assert swept
                    deep.append(any(multi in x for x in swept))
                assert deep[1:] == [False] * 3, (plan.variant_name(v), name, deep)
                seen += deep[0]
        assert seen > 0


def long_lists_without_allocation(h):
    """stencil_run_noalloc takes every list whose offsets and position groups (16 bytes a point) fit its 8 MiB,
    at the sweeps by strips and bricks too, and refuses more."""
    S = h.S
    for kind, shape in ((S.WAVE2, (1100, 1000)), (S.HEAT, (1100, 1000)), (S.WAVE2, (110, 100, 100)),
                        (S.HEAT, (110, 100, 100))):
        w = S.heat_weights(4, 0.05) if kind == S.HEAT else S.second_derivative_weights(4)
        plan = S.Plan(kind, shape, 2, w)
        plan.variant = 0
        f = h.fields(plan, 3 if kind == S.WAVE2 else 2)
        for n, fits in ((1000, True), (300000, True), (522000, True), (1 << 20, False)):
            pos = _points(h, shape, n)
            for src, rec in ((S.Source(n, C.cast(pos, C.c_void_p), C.c_void_p(4096), None), None),
                             (None, S.Receivers(n, C.cast(pos, C.c_void_p), C.c_void_p(8192)))):
                st, _ = h.run(plan, f, 3, src=src, rec=rec, name="stencil_run_noalloc")
                got = [x[0] for x in h.launches()]
                assert (st == 0) == fits, (kind, shape, n, bool(src), st, h.lib.stencil_last_error())
                if st == 0:
                    assert sum("k_step2d" in x or "k_zbrick" in x for x in got) == 3


def batch_variants(h):
    """Each batch variant launches the kernel that it is called after; small batches start with the bricks."""
    S = h.S
    for sides, default in (([(20, 24, 28), (36, 40, 44)], "bricks_64x16x2_t256"),
                           ([(20, 24, 28), (300, 300, 300)], "zmarch_64x32_t256_zc64")):
        batch = S.BatchPlan(sides, 4, S.second_derivative_weights(8))
        names = [batch.variant_name(v) for v in range(batch.variant_count())]
        assert len(set(names)) == len(names) and batch.variant_name(batch.variant) == default
        f = [h.take(layout.bytes) for layout in batch.layouts for _ in range(3)]
        for v, name in list(enumerate(names))[1:]:
            if name.startswith(("tb2_", "persistent_", "shots_")):
                continue
            batch.variant = v
            h.launches()
            assert _run_batch(h, batch, f, 2)[0] == 0
            got = {x[0] for x in h.launches()}
            assert len(got) == 1 and ("k_zbrick_batch" in got.pop()) == name.startswith("bricks_"), name


def saved_choices(h):
    """A choice that an earlier generation of kernels saved is tuned again; one of this generation is taken."""
    S, path = h.S, os.environ["STENCIL_TUNE_CACHE"]

    def tuned():
        plan = S.Plan(S.WAVE2, (40, 44, 48), 4, S.second_derivative_weights(8))
        f = h.fields(plan, 3)
        assert h.lib.stencil_tune(plan.handle, (C.c_void_p * 3)(*f), 1, None) == 0
        return plan.variant_name(plan.variant)

    with open(path, "w") as out:
        out.write("unknown b0:k1:d3:r4:h4:bc0:t0:damp0:40:44:48:B%d zmarch_64x32_t256_zc32\n" % S.Plan(
            S.WAVE2, (40, 44, 48), 4, S.second_derivative_weights(8)).layout.bytes)
    first = tuned()
    assert first != "zmarch_64x32_t256_zc32"
    with open(path) as lines:
        arch, key, name = lines.read().splitlines()[-1].split()
    assert name == first and ":g" in key
    h.launches()
    assert tuned() == first and not h.launches()   # taken without timing


def a_second_device(h):
    """What is asked of the device once (large LDS, the waves it holds) is asked on each device."""
    S = h.S
    grids = []
    for device in (0, 1, 0):
        h.hip.stand_in_device(device)
        plan = S.Plan(S.WAVE2, (40, 44, 48), 4, S.second_derivative_weights(8))
        f, need = h.fields(plan, 3), 0
        for v in range(plan.variant_count()):
            plan.variant = v
            need = plan.run_workspace_bytes()
            if need:
                S.call("stencil_set_workspace", plan.handle, C.c_void_p(h.take(need)), need, None)
            assert h.run(plan, f, 8)[0] == 0
        heat = S.Plan(S.HEAT, (8192, 8192), 4, S.heat_weights(8, 0.05))
        h.launches()
        assert h.run(heat, h.fields(heat, 2), 8)[0] == 0
        swept = [x for x in h.launches() if "k_march2d" in x[0]]
        assert swept
        grids.append(swept[0][1])
    assert grids[1] < grids[0] == grids[2]   # fewer waves at once: longer chunks of rows


def passes_by_size(h):
    """On which side of each line a 2D plan takes several steps per launch, by kind, storage and radius."""
    S = h.S
    w = lambda kind, r: S.heat_weights(2 * r, 0.05) if kind == S.HEAT else S.second_derivative_weights(2 * r)
    for kind, dtype, r, below, above in (
            (S.HEAT, S.F32, 1, 1000, 1200), (S.HEAT, S.F32, 2, 2600, 2802), (S.HEAT, S.F32, 3, 5300, 5600),
            (S.HEAT, S.F32, 4, 5700, 5900), (S.WAVE2, S.F32, 1, 1100, 1302), (S.WAVE2, S.F32, 2, 1900, 2002),
            (S.WAVE2, S.F32, 3, 2500, 2602), (S.WAVE2, S.F32, 4, 4400, 4602), (S.HEAT, S.BF16, 1, 2800, 3002),
            (S.HEAT, S.F16, 2, 7700, 8000), (S.HEAT, S.F16, 3, 15000, 0), (S.HEAT, S.BF16, 4, 15000, 0),
            (S.WAVE2, S.F16, 1, 2400, 2500), (S.WAVE2, S.BF16, 2, 4000, 4202), (S.WAVE2, S.F16, 3, 6600, 6800),
            (S.WAVE2, S.F16, 4, 7800, 8000)):
        for n, deep in ((below, False), (above, True)):
            if n == 0:
                continue
            plan = S.Plan(kind, (n, n), r, w(kind, r), dtype=dtype)
            plan.variant = 0
            f, need = h.fields(plan, 3 if kind == S.WAVE2 else 2), plan.run_workspace_bytes()
            assert need == 0 or kind == S.WAVE2
            if need:
                S.call("stencil_set_workspace", plan.handle, C.c_void_p(h.take(need)), need, None)
            assert need > 0 or not deep or kind == S.HEAT
            h.launches()
            assert h.run(plan, f, 16)[0] == 0
            assert any("k_march2d" in x[0] for x in h.launches()) == deep, (kind, dtype, r, n)


def brick_forms(h):
    """Planes per brick by box, kind, storage and radius (the kernel's last two parameters but one)."""
    S = h.S
    wave, heat = S.WAVE2, S.HEAT
    for kind, dtype, r, shape, planes in (
            (wave, S.F32, 4, (9, 271, 270), 2), (wave, S.F32, 4, (9, 1931, 1953), 4), (wave, S.F32, 2, (23, 1001, 1003), 4),
            (wave, S.F32, 1, (256, 256, 256), 2), (wave, S.F16, 4, (9, 531, 1101), 4), (wave, S.F16, 3, (9, 531, 1101), 2),
            (wave, S.BF16, 4, (20, 40, 80), 2), (wave, S.BF16, 2, (320, 320, 320), 4), (heat, S.F32, 4, (160, 160, 160), 4),
            (heat, S.F32, 3, (128, 128, 128), 2), (heat, S.F32, 2, (160, 160, 160), 2), (heat, S.F16, 1, (160, 160, 160), 4)):
        w = S.heat_weights(2 * r, 0.05) if kind == heat else S.second_derivative_weights(2 * r)
        plan = S.Plan(kind, shape, r, w, dtype=dtype)
        plan.variant = 0
        h.launches()
        assert h.run(plan, h.fields(plan, 3 if kind == wave else 2), 1)[0] == 0
        (name, grid, _), = h.launches()
        tiles = -(-shape[2] // 64) * -(-shape[1] // 16)
        assert "k_zbrick" in name and "Li%dELb0" % planes in name and grid == tiles * -(-shape[0] // planes), (name, shape)


if __name__ == "__main__":
    globals()[sys.argv[2]](Host(sys.argv[1]))
    print("ok")
