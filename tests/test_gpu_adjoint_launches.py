"""The launches of the adjoint: up to 2,048 pairs in groups of 64 lanes, all
configurations in one launch; more pairs in groups of 32 and 64 lanes, in one launch
or (from 32,768 tiles on) one per configuration; tiles of long haplotypes apart.  The same
regions in plans of every size, against the oracle with the adjoint's tolerance."""
import numpy as np
import pytest

from gpu_util import binding, say, wl
from test_gpu_adjoint import compare, gpu_grad, oracle_grad

pytestmark = pytest.mark.gpu

LENS = [1, 31, 32, 63, 64, 95, 96, 127, 128, 159, 160, 191, 192, 255, 256, 319]


def region(rng, lens, haps):
    ref = rng.choice(list("ACGT"), size=1800)
    reads = ["".join(ref[s:s + m]) for m, s in zip(lens, rng.integers(0, 60, len(lens)))]
    return reads, ["".join(ref[:n]) for n in haps]


@pytest.mark.parametrize("copies,what", [(1, "wide, one launch"), (40, "one launch"), (900, "a launch per configuration")])
def test_adjoint_launches(copies, what):
    rng = np.random.default_rng(8)
    base = [region(rng, LENS, [40, 100, 333, 401]), region(rng, LENS[4:9], [1400, 1300]), region(rng, [150, 10], [70])]
    fill = [region(rng, [20, 40, 70, 100, 140, 150, 180, 200], [30, 45, 60, 75, 80, 90, 100, 33])]
    prob = wl.from_strings(base + fill * copies, base_q=30)
    one = wl.from_strings(base, base_q=30)
    say(f"adjoint launches: {what}, {prob.num_pairs} pairs")
    u = rng.normal(size=prob.num_pairs)
    ref, _ = oracle_grad(one, u[:one.num_pairs])
    got, _ = gpu_grad(prob, u)
    assert np.all(np.isfinite(got))
    compare(got[:ref.shape[0]], ref, what)
    # copies of a region with the same upstream gradient: the same rows
    again, _ = gpu_grad(prob, np.concatenate([u[:one.num_pairs], np.ones(prob.num_pairs - one.num_pairs)]))
    rows = again[ref.shape[0]:].reshape(copies, -1, 7)
    assert np.array_equal(rows, np.broadcast_to(rows[:1], rows.shape))
