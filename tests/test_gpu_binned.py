"""The binned launches on problems that are small for the oracle.  A batch of 776 pairs
of 256-base reads beside them, more than the one-pair launch takes, sends a plan and a
call without one to the bins, which every test of a plan asserts: graph replays, length
splits, chains, the FP64 queues, the Viterbi score and explicit parameters, and the
device's own sorting of a call without a plan.  At the end the one-pair launch in the
forms that hold reads of up to 255 bases and longer ones."""
import numpy as np
import pytest

from gpu_util import binding, check_against_oracle, oracle, say, wl
from test_gpu_chains import _chain_problem
from test_gpu_one_pair import LONG, SHORT, problem, same
from test_gpu_parity import RAGGED_M, RAGGED_N, _ragged
from test_zz_no_alloc import _same

pytestmark = pytest.mark.gpu


def concat(*probs):
    cat = lambda f: np.concatenate([getattr(p, f) for p in probs])
    off = lambda f: np.concatenate([[0], np.cumsum(np.concatenate([np.diff(getattr(p, f)) for p in probs]))])
    return wl.Problem(off("batch_read_begin"), off("batch_hap_begin"), off("read_offset"), cat("read_bases"),
                      cat("base_qual"), cat("ins_qual"), cat("del_qual"), cat("gcp_qual"), off("hap_offset"),
                      cat("hap_bases"))


def with_bulk(prob):
    ref = "".join(np.random.default_rng(1).choice(list("ACGT"), size=330))
    return concat(prob, wl.from_strings([([ref[20:276]] * 97, [ref[h:h + 300] for h in range(8)])], base_q=30))


def params(prob, seed, spread=0.1):
    par = oracle.params_from_phred(prob.base_qual, prob.ins_qual, prob.del_qual, prob.gcp_qual)
    par = par * 10 ** np.random.default_rng(seed).uniform(-spread, spread, par.shape)
    return np.log10(par).astype(np.float32)


def run(prob, viterbi=False, lp=None, calls=1, **kw):
    """Scores and statuses of prob, with the bulk batch beside it, through a plan that
    sweeps bins; every call of several into the same buffers, with other work between."""
    import torch
    full = with_bulk(prob)
    if lp is not None:
        lp = torch.from_numpy(np.concatenate([lp, params(full, 3)[len(lp):]])).cuda()
    dev, plan = binding.DeviceProblem(full), binding.Plan(full, **kw)
    out = torch.zeros(full.num_pairs, dtype=torch.float64, device="cuda")
    st = torch.zeros(full.num_pairs, dtype=torch.uint8, device="cuda")
    first = None
    for _ in range(calls):
        out.zero_()
        (plan.viterbi if viterbi else plan.forward)(dev, lp, out=out, status=st)
        x = torch.randn(1 << 18, device="cuda")
        (x * 2).sum().item()
        res = out.cpu().numpy().copy(), st.cpu().numpy().copy()
        assert first is None or (np.array_equal(first[0], res[0]) and np.array_equal(first[1], res[1]))
        first = res
    assert plan.stage_ms()[0] > 0  # binned
    assert plan.rescued() == int((first[1] != binding.PAIR_FP32).sum())
    plan.close()
    if lp is None:  # (explicit parameters differ from read to read)
        bulk = first[0][prob.num_pairs:].reshape(97, 8)
        assert np.abs(bulk - bulk[:1]).max() <= 1e-5
    return first[0][:prob.num_pairs], first[1][:prob.num_pairs]


def ragged(seed, related=True):
    ms, ns = RAGGED_M, RAGGED_N
    prob = _ragged(seed, [ms[:9], ms[9:18], ms[18:], [1], [], [5, 7]], [ns[:6], ns[5:12], ns[11:], [1], [10, 20], []],
                   related=related)
    # a row outside the rescaled states in some reads
    for r in (3, 12, 20):
        o = prob.read_offset[r]
        if prob.read_offset[r + 1] - o > 9:
            prob.ins_qual[o + 7], prob.ins_qual[o + 8] = 2, 90
    return prob


@pytest.mark.parametrize("related", [True, False])
def test_ragged(related):
    prob = ragged(71, related)
    ref, best = oracle.forward(prob), oracle.viterbi(prob)
    say(f"binned, {prob.num_pairs} ragged pairs, log10 L {ref.min():.0f} to {ref.max():.0f}")
    graph = run(prob, calls=4)
    check_against_oracle(prob, *graph, ref=ref)
    direct = run(prob, use_graph=False)
    assert np.array_equal(graph[0], direct[0]) and np.array_equal(graph[1], direct[1])
    check_against_oracle(prob, *run(prob, viterbi=True, calls=4), ref=best)
    forced = run(prob, rescue_threshold=float("inf"))
    assert np.all(forced[1] != binding.PAIR_FP32)
    check_against_oracle(prob, *forced, ref=ref)
    lp = params(prob, 5)
    check_against_oracle(prob, *run(prob, lp=lp, calls=4), log10_params=lp)
    check_against_oracle(prob, *run(prob, viterbi=True, lp=lp), ref=oracle.viterbi(prob, log10_params=lp))


def test_haplotype_length_splits(tmp_path):
    ns = [100, 255, 256, 257, 1008, 1023, 1024, 2047, 2048, 2049, 2176]
    prob = _ragged(61, [[240, 247, 255], [250, 200], [255]], [ns[:6], ns[5:], [2048, 2047]])
    ref = oracle.forward(prob)
    split = tmp_path / "split.txt"
    split.write_text("223 16 14\n255 16 16 256 32 8\n1023 64 16\n")
    for kw in (dict(), dict(tune_table=str(split), calls=3), dict(tune_table=str(split), use_graph=False)):
        check_against_oracle(prob, *run(prob, **kw), ref=ref)
    check_against_oracle(prob, *run(prob, viterbi=True, tune_table=str(split)), ref=oracle.viterbi(prob))


def test_chains():
    for seed, related in ((5, True), (6, False)):
        prob = _chain_problem(seed, related=related)
        ref = oracle.forward(prob)
        got = run(prob, calls=3)
        say(f"chains: {int((got[1] == binding.PAIR_FP64).sum())} of {prob.num_pairs} pairs in FP64")
        assert related or (got[1] == binding.PAIR_FP64).sum() > prob.num_pairs // 2
        check_against_oracle(prob, *got, ref=ref)
        check_against_oracle(prob, *run(prob, viterbi=True), ref=oracle.viterbi(prob))
    prob = _chain_problem(8)
    lp = params(prob, 9, 0.3)
    check_against_oracle(prob, *run(prob, lp=lp), log10_params=lp)


def test_chain_results_inside_a_larger_problem():
    a = _chain_problem(10)
    other = _chain_problem(11)
    one, st = run(a)
    both, sb = run(concat(other, a))
    assert np.array_equal(st, sb[other.num_pairs:])
    assert np.array_equal(one.view(np.int64), both[other.num_pairs:].view(np.int64))


@pytest.mark.parametrize("explicit", [False, True])
@pytest.mark.parametrize("related", [True, False])
def test_without_a_plan(related, explicit):
    """Every bin of the built-in table, reads over 511 bases, both FP64 queues, with and
    without explicit parameters, twice with a smaller problem in between."""
    import torch
    prob = concat(ragged(81, related), wl.config3(pairs=30))
    full = with_bulk(prob)
    lp = params(full, 13) if explicit else None
    tlp = None if lp is None else torch.from_numpy(lp).cuda()
    dev = binding.DeviceProblem(full)
    plan = binding.Plan(full, tune_table="builtin")
    out, st = plan.forward(dev, tlp)
    torch.cuda.synchronize()
    assert plan.stage_ms()[0] > 0  # a call without a plan has the same bound on its long pairs
    want = out.cpu().numpy(), st.cpu().numpy()
    plan.close()
    small = wl.config0()
    sdev = binding.DeviceProblem(small)
    for _ in range(2):
        free, sf = binding.forward_noalloc(full, dev, tlp)
        torch.cuda.synchronize()
        got = free.cpu().numpy(), sf.cpu().numpy()
        _same(full, got, want)
        k = prob.num_pairs
        check_against_oracle(prob, got[0][:k], got[1][:k], log10_params=None if lp is None else lp[:len(prob.read_bases)])
        binding.forward_noalloc(small, sdev)
    assert (got[1] == binding.PAIR_FP64).sum() >= 10


@pytest.mark.parametrize("lens,repeat,launches", [
    (SHORT + LONG, 4, 2),       # 1,623 pairs, 540 of them long, reads of up to 1,023 bases
    (SHORT + LONG[:3], 14, 2),  # 4,413 pairs, 630 long, up to 320 bases
    (SHORT + LONG[:4], 1, 1)])  # 333 pairs, up to 447 bases
def test_one_pair_short_and_long(lens, repeat, launches):
    import torch
    prob = problem(lens, seed=33, repeat=repeat)
    long_pairs = int((prob.read_lengths[prob.pair_index()[0]] > 255).sum())
    assert long_pairs <= 768 and (prob.num_pairs > (768 if max(lens) > 511 else 4096)) == (launches == 2)
    dev = binding.DeviceProblem(prob)
    plan = binding.Plan(prob, tune_table=binding.TUNED_TABLE)
    bins = binding.Plan(prob, tune_table=binding.TUNED_TABLE, single_launch=True)
    res = {}
    for name, f in (("one", plan.forward), ("bins", bins.forward), ("one v", plan.viterbi), ("bins v", bins.viterbi)):
        out, st = f(dev)
        torch.cuda.synchronize()
        res[name] = out.cpu().numpy(), st.cpu().numpy()
        if f in (plan.forward, plan.viterbi):
            assert plan.stage_ms()[0] == 0 and plan.rescued() == int((res[name][1] != binding.PAIR_FP32).sum())
    assert bins.stage_ms()[0] > 0
    say(f"one-pair, {launches} launches: {prob.num_pairs} pairs, statuses {np.bincount(res['one'][1], minlength=3).tolist()}")
    same(res["one"], res["bins"], "forward")
    same(res["one v"], res["bins v"], "viterbi")
    pairs = np.sort(np.random.default_rng(2).choice(prob.num_pairs, 300, replace=False))
    check_against_oracle(prob, *res["one"], pairs=pairs)
    free, sf = binding.forward_noalloc(prob, dev)
    torch.cuda.synchronize()
    _same(prob, (free.cpu().numpy(), sf.cpu().numpy()), res["one"])
    plan.close()
    bins.close()
