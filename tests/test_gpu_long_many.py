"""Plans with many long pairs (more than 3,072 windows of 256 rows): one window of
16 rows per lane (FP32) or 4 (FP64) per workgroup, every boundary handed on through
memory.  Forward, Viterbi score and explicit parameters, FP32 and FP64, at the edges
of both window sizes and of the 64 columns that are handed on at a time, against the
oracle and against a plan with few of the pairs, whose windows share workgroups."""
import numpy as np
import pytest

from gpu_util import binding, check_against_oracle, gpu_forward, gpu_viterbi, oracle, say, wl

pytestmark = pytest.mark.gpu

READS = [1024, 1279, 1280, 1535, 1536, 2047, 2048, 2049]
HAPS = [1, 62, 63, 64, 65, 127, 128, 129, 1500]
FEW_ITEMS = 3072  # windows of 256 rows


@pytest.fixture(scope="module")
def problems():
    rng = np.random.default_rng(41)
    ref = rng.choice(list("ACGT"), size=2600)

    def read(m):
        r = ref[20:20 + m].copy()
        err = rng.random(m) < 0.002
        r[err] = rng.choice(list("ACGTN"), size=int(err.sum()))
        return "".join(r)

    reads, haps = [read(m) for m in READS], ["".join(ref[:n]) for n in HAPS]
    few = [(reads, haps)]
    many = few + [(reads[:1], haps[:5])] * 120
    windows = lambda b: sum(len(hs) * (len(r) // 256 + 1) for rs, hs in b for r in rs)
    assert windows(few) <= FEW_ITEMS < windows(many)
    few, many = wl.from_strings(few, base_q=37), wl.from_strings(many, base_q=37)
    return few, many


def same_as_few(few, many, name):
    (gf, sf), (gm, sm) = few, many
    k = len(gf)
    assert np.array_equal(sf, sm[:k]), name
    fp32, fp64 = sf == binding.PAIR_FP32, sf == binding.PAIR_FP64
    assert np.array_equal(gf[fp32], gm[:k][fp32]), name
    assert not fp64.any() or np.abs(gf[fp64] - gm[:k][fp64]).max() <= 1e-9, name
    # copies of a pair have the same score
    rest = gm[k:].reshape(120, -1)
    assert np.array_equal(rest, np.broadcast_to(rest[:1], rest.shape)), name


@pytest.mark.parametrize("threshold", [None, float("inf")])
@pytest.mark.parametrize("viterbi", [False, True])
def test_many_long_pairs(problems, viterbi, threshold):
    few, many = problems
    run, exact = (gpu_viterbi, oracle.viterbi) if viterbi else (gpu_forward, oracle.forward)
    name = f"viterbi={viterbi} threshold={threshold}"
    say(f"many long pairs: {name}")
    f, m = run(few, rescue_threshold=threshold), run(many, rescue_threshold=threshold)
    if threshold:
        assert np.all(m[1] != binding.PAIR_FP32)
    check_against_oracle(few, m[0][:few.num_pairs], m[1][:few.num_pairs], ref=exact(few))
    same_as_few(f, m, name)


def test_many_long_pairs_explicit_parameters(problems):
    few, many = problems
    say("many long pairs: explicit parameters")

    def params(prob):
        par = oracle.params_from_phred(prob.base_qual, prob.ins_qual, prob.del_qual, prob.gcp_qual)
        i = np.arange(len(par))[:, None]
        own = np.concatenate([np.arange(m) for m in np.diff(prob.read_offset)])[:, None]
        assert len(own) == len(i)
        par = par * 10 ** (0.04 * np.sin(0.37 * own + np.arange(7)))
        # a row outside the rescaled states in the first window of one read
        par[prob.read_offset[2] + 300, 0] = 0.0
        with np.errstate(divide="ignore"):
            return np.log10(par).astype(np.float32)

    lf, lm = params(few), params(many)
    f, m = gpu_forward(few, log10_params=lf), gpu_forward(many, log10_params=lm)
    check_against_oracle(few, m[0][:few.num_pairs], m[1][:few.num_pairs], log10_params=lf)
    same_as_few(f, m, "explicit")
    assert np.all(m[1][2 * len(HAPS):3 * len(HAPS)] != binding.PAIR_FP32)
