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


@pytest.mark.parametrize("what", ["forward", "viterbi", "backward"])
def test_calls_with_other_buffers_do_not_wait(what):
    """Buffers that change from call to call, as autograd's do: no call waits for the one
    before it, whether that one replayed a graph or not, and every result is the
    direct launches'."""
    import torch
    prob = wl.config1(regions=200) if what != "backward" else wl.config4(pairs=2500)
    dev = binding.DeviceProblem(prob)
    P, bases = prob.num_pairs, int(prob.read_offset[-1])
    u = torch.linspace(0.5, 1.5, P, dtype=torch.float64, device="cuda")

    def buffers():
        if what == "backward":
            return dict(grad_params=torch.zeros((bases, 7), device="cuda"))
        return dict(out=torch.zeros(P, dtype=torch.float64, device="cuda"),
                    status=torch.zeros(P, dtype=torch.uint8, device="cuda"))

    def call(plan, kw):
        plan.backward(dev, u, **kw) if what == "backward" else getattr(plan, what)(dev, **kw)

    direct = binding.Plan(prob, use_graph=False, keep_checkpoints=True)
    want = buffers()
    call(direct, want)
    torch.cuda.synchronize()
    assert what == "backward" or binned(direct)
    direct.close()
    plan = binding.Plan(prob, keep_checkpoints=True)
    a, b, c = buffers(), buffers(), buffers()
    waited = []
    for kw in (a, b, a, a, a, b, a, b, b, b, c, c, a, b, c):
        for t in kw.values():
            t.zero_()
        call(plan, kw)
        torch.cuda.synchronize()
        for k, t in kw.items():
            assert torch.equal(t, want[k])
    # without a wait between the calls: each returns before the one before it has run
    done = None
    for kw in (a, a, b, b, b, c, a, a):
        busy(10)
        call(plan, kw)
        if done:
            waited.append(done.query())
        done = torch.cuda.Event()
        done.record()
    torch.cuda.synchronize()
    for kw in (a, b, c):
        for k, t in kw.items():
            assert torch.equal(t, want[k])
    say(f"{what}: {sum(waited)} of {len(waited)} calls waited")
    assert not any(waited)
    plan.close()


def test_training_steps_through_a_default_plan():
    """Steps of learning the parameters: a default plan's log-likelihoods and gradients
    are a direct plan's, bit for bit, and no step waits for the one before."""
    import torch
    from paper_2411_11547_amd.autograd import pairhmm_log10_likelihood
    prob = wl.config4(pairs=600)
    dev = binding.DeviceProblem(prob)
    p = {f: torch.from_numpy(10.0 ** (getattr(prob, f).astype(np.float64) / -10.0)).cuda()
         for f in ("base_qual", "ins_qual", "del_qual", "gcp_qual")}
    q, de, ze, ep = (p[f] for f in ("base_qual", "ins_qual", "del_qual", "gcp_qual"))
    start = torch.log10(torch.stack([1 - de - ze, 1 - ep, de, ep, ze, 1 - q, q / 3], 1)).float()

    def steps(plan, wait):
        x, out, done = start.clone().requires_grad_(True), [], None
        for _ in range(6):
            if wait is not None:
                busy(10)
            x.grad = None
            ll = pairhmm_log10_likelihood(x, plan, dev)
            ll.sum().backward()
            if wait is not None:  # the step before
                if done:
                    wait.append(done.query())
                done = torch.cuda.Event()
                done.record()
            out.append((ll.detach().clone(), x.grad.clone()))
            with torch.no_grad():
                x -= 1e-4 * x.grad
        torch.cuda.synchronize()
        return out

    # (keep_checkpoints: a plan's first backward call builds the adjoint's tables)
    one, two = binding.Plan(prob, keep_checkpoints=True), binding.Plan(prob, use_graph=False, keep_checkpoints=True)
    steps(one, None)  # memory for parameters and gradients is there
    waited = []
    got, want = steps(one, waited), steps(two, None)
    for (la, ga), (lb, gb) in zip(got, want):
        assert torch.equal(la, lb) and torch.equal(ga, gb)
    say(f"{len(got)} steps, {sum(waited)} waited")
    assert not any(waited)
    one.close()
    two.close()


def test_default_plan_inside_a_captured_graph():
    """A caller's own graph around a default plan's calls, replayed with other work and
    other inputs in between."""
    import torch
    prob = wl.config1(regions=200)
    dev = binding.DeviceProblem(prob)
    plan = binding.Plan(prob)
    P = prob.num_pairs
    out = torch.zeros(P, dtype=torch.float64, device="cuda")
    st = torch.zeros(P, dtype=torch.uint8, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for _ in range(3):
            plan.forward(dev, out=out, status=st)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        plan.forward(dev, out=out, status=st)
    quals = dev.t["base_qual"].clone()
    for k in range(4):
        dev.t["base_qual"].copy_(quals - (k % 2) * 3)
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        got = out.clone()
        other = torch.empty_like(out)
        plan.forward(dev, out=other, status=st)
        torch.cuda.synchronize()
        assert torch.equal(got, other), k
    plan.close()


def test_plan_destroyed_after_a_captured_call():
    """A call inside a caller's capture takes the plan's events with it: a plan that is
    destroyed then still waits for the graph that its call before the capture replays."""
    import torch
    prob = wl.config1(regions=200)
    ref, rst = gpu_forward(prob, use_graph=False)
    dev = binding.DeviceProblem(prob)
    plan = binding.Plan(prob)
    out = torch.zeros(prob.num_pairs, dtype=torch.float64, device="cuda")
    st = torch.zeros(prob.num_pairs, dtype=torch.uint8, device="cuda")
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        plan.forward(dev, out=out, status=st)
        assert binned(plan)
        out.zero_()
        busy()
        plan.forward(dev, out=out, status=st)
        g.capture_begin(capture_error_mode="relaxed")
        plan.forward(dev, out=out, status=st)
        g.capture_end()
        plan.close()
        assert side.query()
    assert np.array_equal(st.cpu().numpy(), rst) and np.array_equal(out.cpu().numpy(), ref)
