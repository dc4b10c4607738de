"""Plans that capture their launches (use_graph, the default) in a program that does
not wait between calls."""
import numpy as np
import pytest

from gpu_util import binding, gpu_forward, say, wl

pytestmark = pytest.mark.gpu


def binned(plan):
    return plan.stage_ms()[0] > 0


def busy(ms=30.0):
    """GPU work of about that length on the current stream, so that what is enqueued
    after it is still to run when the host goes on."""
    import torch
    torch.cuda._sleep(int(ms * 1e6 * 2))


def test_plan_destroyed_while_its_graph_runs():
    """A plan that goes away right after its call (a temporary one in a program that
    reads the scores later): its graphs are waited for before they are destroyed."""
    import torch
    prob = wl.config1(regions=200)
    ref, rst = gpu_forward(prob, use_graph=False)
    dev = binding.DeviceProblem(prob)
    outs = []
    for _ in range(4):
        plan = binding.Plan(prob)
        out = torch.empty(prob.num_pairs, dtype=torch.float64, device="cuda")
        st = torch.empty(prob.num_pairs, dtype=torch.uint8, device="cuda")
        for _ in range(2):
            plan.forward(dev, out=out, status=st)
        assert binned(plan)
        busy()
        plan.forward(dev, out=out, status=st)
        plan.close()
        outs.append((out, st))
    torch.cuda.synchronize()
    say(f"{len(outs)} plans destroyed with a call under way")
    for out, st in outs:
        assert np.array_equal(st.cpu().numpy(), rst) and np.array_equal(out.cpu().numpy(), ref)
