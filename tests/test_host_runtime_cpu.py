"""The library's host code without a GPU: what it launches, captures, replays
and keeps, on the stand-in HIP calls of hip_stand_in.cpp (checks in
_host_runtime.py, each in a process of its own)."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ is not available")
    lib = str(tmp_path_factory.mktemp("hip") / "libhip_stand_in.so")
    subprocess.run([gxx, "-std=c++17", "-O1", "-fPIC", "-shared", "-Wall", "-o", lib,
                    os.path.join(HERE, "hip_stand_in.cpp")], check=True)
    return lib


@pytest.mark.parametrize("check", ["shrunk_workspace", "concurrent_batch", "runs_that_are_not_repeated", "runs_in_a_caller_capture",
                                   "heat_points", "long_lists_without_allocation", "batch_variants",
                                   "saved_choices", "a_second_device",
                                   "passes_by_size", "brick_forms"])
def test_host_runtime(stand_in, check, tmp_path):
    r = subprocess.run([sys.executable, os.path.join(HERE, "_host_runtime.py"), stand_in, check], capture_output=True,
                       text=True, timeout=300, env=dict(os.environ, STENCIL_TUNE_CACHE=str(tmp_path / "tuned")))
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), (r.stdout + r.stderr)[-4000:]


def test_a_short_memory_declines_only_an_optional_workspace(monkeypatch):
    import torch

    import paper_2404_02218_amd as S
    asked = []

    def empty(n, **kw):
        asked.append(n)
        raise torch.cuda.OutOfMemoryError("out of memory")

    monkeypatch.setattr(torch, "empty", empty)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    wave2d = S.Plan(S.WAVE2, (3000, 3013), 4, S.second_derivative_weights(8))
    wave3d = S.Plan(S.WAVE2, (40, 44, 48), 4, S.second_derivative_weights(8))
    wave3d.variant = 21   # two steps per pass, which needs its field pair
    for _ in range(3):
        wave2d._ws.ensure(wave2d.handle, optional=True)
    assert asked == [wave2d.run_workspace_bytes()] and asked[0] > 0   # asked for once, then done without
    with pytest.raises(torch.cuda.OutOfMemoryError):
        wave3d._ws.ensure(wave3d.handle)
