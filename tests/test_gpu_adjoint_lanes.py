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
