"""The adjoint of small plans in groups of 32 and of 64 lanes, by the rule's sides:
reads of one row per lane beside longer ones, plans of one configuration with more and
fewer than 1,024 pairs, against the oracle with the adjoint's tolerance."""
import numpy as np
import pytest

from gpu_util import binding, say, wl
from test_gpu_adjoint import compare, gpu_grad, oracle_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,haps,copies", [
    ([31, 1, 30, 31], [40, 70, 300], 90),             # one row per lane, 1,080 pairs
    ([63, 40, 32, 33], [300, 299, 250], 20),          # two rows of 32 lanes: 240 pairs, 64 lanes
    ([63, 40, 32, 33], [300, 299, 250], 90),          # 1,080 pairs, 32 lanes
    ([127, 100, 96, 120], [1000, 990, 64], 90),       # 64 lanes
    ([159, 150, 128, 140], [1400, 1300, 1390], 90),   # 32 lanes, long haplotypes
    ([31, 32, 5, 200, 319, 150], [90, 333, 1290], 30)])  # several configurations
def test_small_plans(lens, haps, copies):
    rng = np.random.default_rng(len(haps) + sum(lens))
    ref = rng.choice(list("ACGT"), size=1500)
    reads = ["".join(ref[s:s + m]) for m, s in zip(lens, rng.integers(0, 40, len(lens)))]
    one = wl.from_strings([(reads, ["".join(ref[:n]) for n in haps])], base_q=30)
    prob = wl.from_strings([(reads, ["".join(ref[:n]) for n in haps])] * copies, base_q=30)
    say(f"adjoint: reads {lens}, haplotypes {haps}, {prob.num_pairs} pairs")
    assert prob.num_pairs <= 2048
    u = rng.normal(size=one.num_pairs)
    ref_grad, _ = oracle_grad(one, u)
    got, _ = gpu_grad(prob, np.tile(u, copies))
    assert np.all(np.isfinite(got))
    compare(got[:ref_grad.shape[0]], ref_grad, "small plan")
    rows = got.reshape(copies, -1, 7)
    assert np.array_equal(rows, np.broadcast_to(rows[:1], rows.shape))


@pytest.mark.parametrize("copies", [1, 260])
def test_long_haplotypes_beside_short_ones(copies):
    """Haplotypes around the steps that part the groups of tiles (1,280, 2,560, 5,120) and
    a very long one, in one launch (few pairs) and, where its LDS and its slice would
    leave few workgroups for many other pairs, in launches of their own."""
    rng = np.random.default_rng(11)
    ref = rng.choice(list("ACGT"), size=20000)
    cut = lambda m, s: "".join(ref[s:s + m])
    base = [([cut(100, 30)], [cut(20000, 0)]),
            ([cut(m, 5) for m in (150, 140, 90, 31)], [cut(n, 0) for n in (1247, 1248, 2527, 2528)]),
            ([cut(200, 9), cut(319, 9)], [cut(n, 0) for n in (1215, 1216, 5055, 5056)])]
    fill = [([cut(m, 7) for m in (40, 60, 90, 100, 130, 150, 159, 160, 200, 230, 250, 300, 310, 70, 80, 110, 120, 155, 170, 190)],
             [cut(n, 0) for n in (420, 440, 460, 480, 500)])]
    prob, one = wl.from_strings(base + fill * copies, base_q=30), wl.from_strings(base + fill, base_q=30)
    say(f"adjoint: {prob.num_pairs} pairs, haplotypes of 420 to 20,000 bases")
    u = rng.normal(size=one.num_pairs)
    of_fill = u[-100:]
    want, _ = oracle_grad(one, u)
    got, _ = gpu_grad(prob, np.concatenate([u, np.tile(of_fill, copies - 1)]))
    compare(got[:want.shape[0]], want, "long haplotypes")
    rows = got[-copies * sum(len(r) for r in fill[0][0]):].reshape(copies, -1, 7)
    assert np.array_equal(rows, np.broadcast_to(rows[:1], rows.shape))


@pytest.mark.parametrize("n,ok", [(25600, True), (25984, False), (40000, False)])
@pytest.mark.parametrize("copies", [1, 3000])
def test_longest_haplotype_of_the_adjoint(n, ok, copies):
    """The longest haplotype that is accepted is the same for few pairs and for many."""
    import torch
    read, hap = "ACGT" * 25, "ACGTTGCA" * (n // 8)
    prob = wl.from_strings([([read], [hap])] + [([read], [hap[:120]])] * copies, base_q=30)
    dev, plan = binding.DeviceProblem(prob), binding.Plan(prob)
    u = torch.ones(prob.num_pairs, dtype=torch.float64, device="cuda")
    if ok:
        got = plan.backward(dev, u)
        torch.cuda.synchronize()
        assert bool(torch.isfinite(got).all())
    else:
        with pytest.raises(binding.PHError) as e:
            plan.backward(dev, u)
        assert e.value.status == -2 and "too long" in str(e.value)
    plan.close()
