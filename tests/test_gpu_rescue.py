"""The FP64 sweeps of the binned launches, class by class of read lengths: pairs that
the rescaled states finish, pairs that they pass on (below 2^-1000 of their scale) to
the plain states, pairs below that range too, and reads with a row that goes to the
plain states at once, against the oracle; the count of pairs sent to FP64."""
import numpy as np
import pytest

from gpu_util import binding, check_against_oracle, oracle, say, wl

pytestmark = pytest.mark.gpu


def stressed(m_lo, m_hi, reads, haps, seed):
    """Reads of m_lo .. m_hi bases with 0 to m / 2.6 mismatches of Phred 40, so that log10 L
    spans every range of the sweeps where the reads are long enough."""
    rng = np.random.default_rng(seed)
    ref = rng.integers(0, 4, m_hi + 60)
    rs = []
    for k, m in enumerate(np.linspace(m_lo, m_hi, reads).astype(int)):
        r = ref[int(rng.integers(0, 40)):][:m].copy()
        at = np.sort(rng.choice(m, int(m * (k % 23) / 22 / 2.6), replace=False))
        r[at] = (r[at] + 1 + rng.integers(0, 3, len(at))) % 4
        rs.append("".join("ACGT"[b] for b in r))
    hs = ["".join("ACGT"[b] for b in ref[:len(ref) - 3 * h]) for h in range(haps)]
    prob = wl.from_strings([(rs, hs)], base_q=40)
    # every 20th read: a gap-open quality that rises from 2 to 90
    for r in range(7, reads, 20):
        prob.ins_qual[prob.read_offset[r] + 9] = 2
        prob.ins_qual[prob.read_offset[r] + 10] = 90
    return prob


@pytest.mark.parametrize("m_lo,m_hi,reads,haps", [(40, 127, 46, 4), (128, 255, 46, 4), (256, 511, 200, 5), (512, 1023, 200, 5)])
@pytest.mark.parametrize("threshold", [None, float("inf")])
@pytest.mark.parametrize("viterbi", [False, True])
def test_rescue_classes(m_lo, m_hi, reads, haps, threshold, viterbi):
    import torch
    prob = stressed(m_lo, m_hi, reads, haps, seed=m_lo)
    dev = binding.DeviceProblem(prob)
    # force_p names a launch: never the one-pair launch
    plan = binding.Plan(prob, rescue_threshold=threshold, force_p=16 if m_hi <= 255 else 64)
    out, st = (plan.viterbi if viterbi else plan.forward)(dev)
    torch.cuda.synchronize()
    assert plan.stage_ms()[0] > 0  # binned
    got, st, sent = out.cpu().numpy(), st.cpu().numpy(), plan.rescued()
    plan.close()
    ref = (oracle.viterbi if viterbi else oracle.forward)(prob)
    say(f"reads {m_lo}-{m_hi}: {prob.num_pairs} pairs, log10 in [{ref.min():.0f}, {ref.max():.0f}], "
        f"statuses {np.bincount(st, minlength=3).tolist()}")
    check_against_oracle(prob, got, st, ref=ref)
    assert sent == int((st != binding.PAIR_FP32).sum())
    assert (st == binding.PAIR_FP64).sum() >= reads * haps // 8
    if m_lo >= 512:  # passed on and finished, and passed on below the range
        assert (st == binding.PAIR_FP64_FLOOR).any()
