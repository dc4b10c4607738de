"""Which calls take the one-pair launch and which the bins: shapes on either side of
the line whose two times lie far apart, each with the results of the oracle and of the
call without a plan."""
import numpy as np
import pytest

from gpu_util import binding, check_against_oracle, oracle, say, wl

pytestmark = pytest.mark.gpu

# regions of 15 reads and 5 haplotypes: read and haplotype bases, regions, one-pair
# launch or not (us of the bins and of the one-pair launch)
SHAPES = [(10, 300, 60, True),       # 62, 47
          (10, 300, 200, False),     # 79, 113
          (30, 1000, 200, False),    # 166, 275
          (60, 300, 60, True),       # 110, 46
          (60, 300, 600, False),     # 227, 302
          (60, 2000, 320, False),    # 480, 800
          (100, 1000, 60, True),     # 169, 133
          (100, 1000, 200, False),   # 278, 352
          (150, 300, 60, True),      # 163, 73
          (250, 300, 200, True)]     # 271, 221


@pytest.mark.parametrize("m,n,regions,one", SHAPES)
def test_route(m, n, regions, one):
    import torch
    rng = np.random.default_rng(m + n)
    ref = rng.choice(list("ACGT"), size=n + 40)
    reads = ["".join(ref[s:s + m]) for s in rng.integers(0, n - m + 1, 15)]
    haps = ["".join(ref[s:s + n]) for s in rng.integers(0, 40, 5)]
    prob = wl.from_strings([(reads, haps)] * regions, base_q=30)
    dev = binding.DeviceProblem(prob)
    plan = binding.Plan(prob)
    out, st = plan.forward(dev)
    torch.cuda.synchronize()
    say(f"{m} x {n}, {prob.num_pairs} pairs: {'one-pair' if plan.stage_ms()[0] == 0 else 'binned'}")
    assert (plan.stage_ms()[0] == 0) == one
    plan.close()
    single = wl.from_strings([(reads, haps)], base_q=30)
    check_against_oracle(single, out[:75].cpu().numpy(), st[:75].cpu().numpy())
    free, sf = binding.forward_noalloc(prob, dev)
    assert torch.equal(sf, st)
    assert float((free - out).abs().max()) <= 1e-5
    # (a tile takes reads of one region, so copies have the same bits)
    assert torch.equal(out.reshape(regions, 75), out[:75].expand(regions, 75))
