"""Runs enqueued directly, captured behind a direct run, captured at the second
call and replayed: the same bits as runs without graphs, whichever way the step
counts, the buffers and the caller's own work alternate."""
import pytest

import paper_2404_02218_amd as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", [S.HEAT, S.WAVE2])
@pytest.mark.parametrize("shape", [(70, 90), (20, 24, 28), (2100, 2050), (162, 162, 162)])   # the last two past 2^22 points
def test_runs_equal_runs_without_graphs(device, monkeypatch, shape, kind):
    import torch
    w = S.heat_weights(4, 0.05) if kind == S.HEAT else S.second_derivative_weights(4)
    inner = (slice(2, -2),) * len(shape)

    def levels(no_graph):
        monkeypatch.setenv("STENCIL_NO_GRAPH", "1" if no_graph else "0")
        plan = S.Plan(kind, shape, 2, w)
        plan.variant = 0
        gen = torch.Generator(device="cuda").manual_seed(3)
        f = [plan.field() for _ in range(3 if kind == S.WAVE2 else 2)]
        f[0].view[inner] = torch.randn(shape, generator=gen, device="cuda")
        if kind == S.WAVE2:
            f[2].view.fill_(0.01)
        out = []
        for k, n in enumerate([3, 3, 4, 4, 4, 2, 4, 4, 1, 4, 3, 3]):
            plan.run(f, n)
            out.append(f[0].view.clone())
            f[0].view[inner] *= 0.5 + 0.1 * (k % 3)   # the caller's own work between runs
        torch.cuda.synchronize()
        return out

    for got, want in zip(levels(False), levels(True)):
        assert torch.equal(got.view(torch.int32), want.view(torch.int32))
