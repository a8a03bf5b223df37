"""GPU: a caller's graph of psatd_step_noalloc and later tuning calls.  The graph
goes on running what it captured, and tuning calls are legal during the capture."""
import pytest

from paper_1707_08500_amd import synth

from psatd_cases import GpuCase, random_fields, say

pytestmark = pytest.mark.gpu


def pair(precision):
    N = (32, 32, 48)
    lo, n, g = synth.uniform_decomposition(N, (2, 2, 3), 4)
    E, B, J = random_fields(N, 81, p=8)
    return [GpuCase(N, lo, n, g, 8, 0.5, 1.0, precision, "replicated", E, B, J) for _ in range(2)]


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_captured_steps_and_tuning(precision):
    """Two captured steps with a tuning call between them, replayed between other
    settings' eager steps on the same plan: every replay equals two eager steps."""
    import torch
    say(f"captured steps and tuning calls, {precision}")
    got, ref = pair(precision)
    plan = got.plan
    plan.step_noalloc(got.E, got.B, got.J)
    plan.sync()
    ref.plan.step(ref.E, ref.B, ref.J)
    default = plan.tuning()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        plan.set_stream(torch.cuda.current_stream().cuda_stream)
        plan.step_noalloc(got.E, got.B, got.J)
        plan.set_tuning(z_threads=1024)
        plan.step_noalloc(got.E, got.B, got.J)
    plan.set_stream(torch.cuda.current_stream().cuda_stream)
    spare = pair(precision)[0]
    for setting in (dict(split_xy=1), dict(batch_boxes=5), dict(fuse_eb=1), dict(z_pencils=4), dict(xy_threads=1024)):
        back = {k: default[k] for k in list(setting) + ["pull_eb"]}
        plan.set_tuning(**setting)
        plan.step(spare.E, spare.B, spare.J)
        graph.replay()
        torch.cuda.synchronize()
        for _ in range(2):
            ref.plan.step(ref.E, ref.B, ref.J)
        ref.plan.sync()
        assert all(torch.equal(a, b) for a, b in zip(got.E + got.B + got.J, ref.E + ref.B + ref.J)), setting
        plan.set_tuning(**back)
