"""The one-pair launch of small calls (one pair per wave, 64 lanes): the same
results, bit for bit, as the binned launches, whose tiles hold several reads and
chains of haplotypes, and within tolerance of the FP64 oracle."""
import numpy as np
import pytest

from gpu_util import binding, check_against_oracle, gpu_forward, gpu_viterbi, oracle, say, wl

pytestmark = pytest.mark.gpu

# edges of the rows per lane (64 lanes, and the 16 lanes of the binned tiles) and of the flush groups
SHORT = [1, 2, 15, 16, 31, 47, 63, 64, 65, 100, 127, 128, 150, 191, 192, 240, 254, 255]
LONG = [256, 319, 320, 447, 511, 512, 700, 1000, 1023]
HAPS = [1, 30, 31, 32, 33, 63, 64, 65, 70, 95, 129, 300, 301, 640]


def problem(read_lens, seed, repeat=4):
    """One batch of `repeat` reads of every length against haplotypes of all
    lengths (so that the binned plan has chain tiles), and one of single pairs."""
    rng = np.random.default_rng(seed)
    ref = rng.choice(list("ACGT"), size=1400)
    reads = []
    for m in read_lens:
        for _ in range(repeat):
            s = int(rng.integers(0, 200))
            r = ref[s:s + m].copy()
            err = rng.random(m) < 0.01
            r[err] = rng.choice(list("ACGTN"), size=int(err.sum()))
            reads.append("".join(r))
    haps = ["".join(ref[int(s):int(s) + n]) for n, s in zip(HAPS, rng.integers(0, 150, len(HAPS)))] + ["".join(ref)]
    prob = wl.from_strings([(reads, haps), (reads[:1], haps[3:5]), (reads[-1:], haps[-1:])])
    prob.base_qual[:] = rng.integers(2, 41, size=len(prob.base_qual))
    prob.ins_qual[:] = rng.integers(20, 46, size=len(prob.ins_qual))
    prob.del_qual[:] = rng.integers(20, 46, size=len(prob.del_qual))
    prob.gcp_qual[:] = 10
    return prob


def same(one, binned, what):
    (go, so), (gb, sb) = one, binned
    assert np.array_equal(so, sb), what
    fp32 = so == binding.PAIR_FP32
    assert np.array_equal(go[fp32], gb[fp32]), (what, np.abs(go - gb)[fp32].max())
    ok = so == binding.PAIR_FP64
    assert not ok.any() or np.abs(go[ok] - gb[ok]).max() <= 1e-9, what  # the same FP64 sweep, other tile order


@pytest.mark.parametrize("lens,force_p", [(SHORT, 16), (LONG, 64)])
def test_one_pair_equals_binned(lens, force_p):
    prob = problem(lens, seed=len(lens))
    one = gpu_forward(prob, tune_table="builtin")  # the same (lanes, rows) per read as force_p
    say(f"{prob.num_pairs} pairs, statuses {np.bincount(one[1], minlength=3).tolist()}")
    check_against_oracle(prob, *one, ref=oracle.forward(prob))
    same(one, gpu_forward(prob, force_p=force_p), "forward")
    same(gpu_viterbi(prob, tune_table="builtin"), gpu_viterbi(prob, force_p=force_p), "viterbi")


@pytest.mark.parametrize("lens", [SHORT, LONG])
def test_one_pair_forced_fp64(lens):
    prob = problem(lens, seed=5, repeat=1)
    got, st = gpu_forward(prob, rescue_threshold=float("inf"))
    assert np.all(st != binding.PAIR_FP32)
    check_against_oracle(prob, got, st)


def test_one_pair_plan_free_and_rescued_count():
    """The plan-free call takes the same launch, with the batches in its arguments
    and (300 batches) on the device: a plan's statuses and FP64 values, and its FP32
    values to rounding (1e-5: a plan groups the row sums as its chains do)."""
    import torch
    for prob in (problem(SHORT + LONG, seed=9, repeat=1),
                 wl.from_strings([(["ACGTNACGGT"[:1 + q % 10] * 9], ["ACGTTACGGT" * (1 + q % 4)]) if q % 7 else ([], ["ACGT"])
                                  for q in range(300)])):
        dev = binding.DeviceProblem(prob)
        plan = binding.Plan(prob, tune_table="builtin")
        out, st = plan.forward(dev)
        torch.cuda.synchronize()
        assert plan.rescued() == int((st != binding.PAIR_FP32).sum())
        assert plan.stage_ms()[1] > 0
        free, sf = binding.forward_noalloc(prob, dev)
        torch.cuda.synchronize()
        assert torch.equal(sf, st)
        fp32 = st == binding.PAIR_FP32
        assert torch.equal(free[~fp32], out[~fp32])
        assert float((free - out)[fp32].abs().max()) <= 1e-5
        plan.close()


@pytest.mark.parametrize("reads,one", [(96, True), (97, False)])
def test_one_pair_limit_of_long_reads(reads, one):
    """768 pairs of reads over 255 bases run at once; one read more takes the bins."""
    rng = np.random.default_rng(4)
    ref = "".join(rng.choice(list("ACGT"), size=400))
    prob = wl.from_strings([([ref[q % 50:][:300] for q in range(reads)], [ref[8 * h:][:330] for h in range(8)])])
    plan = binding.Plan(prob, tune_table="builtin")
    dev = binding.DeviceProblem(prob)
    got, st = plan.forward(dev)
    assert (plan.stage_ms()[0] == 0) == one
    free, sf = binding.forward_noalloc(prob, dev)
    same((got.cpu().numpy(), st.cpu().numpy()), gpu_forward(prob, force_p=64), "forward")
    assert bool((st == sf).all()) and float((free - got).abs().max()) <= 1e-5
    plan.close()


@pytest.mark.parametrize("lens,repeat", [(SHORT + LONG[:5], 2), (SHORT + LONG, 1)])
def test_one_pair_short_and_long_in_one_launch(lens, repeat):
    """Reads up to 255 bases beside reads of up to 511, and of up to 1,023, in one
    launch: the binned launches' results with the same table, FP32 and FP64."""
    prob = problem(lens, seed=21, repeat=repeat)
    assert prob.num_pairs <= 768
    table = dict(tune_table=binding.TUNED_TABLE)
    bins = dict(table, single_launch=True)  # never the one-pair launch; the same (lanes, rows)
    one = gpu_forward(prob, **table)
    check_against_oracle(prob, *one, ref=oracle.forward(prob))
    same(one, gpu_forward(prob, **bins), "forward")
    same(gpu_viterbi(prob, **table), gpu_viterbi(prob, **bins), "viterbi")
    got, st = gpu_forward(prob, rescue_threshold=float("inf"))
    assert np.all(st != binding.PAIR_FP32)
    check_against_oracle(prob, got, st)
