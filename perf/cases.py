"""The work that a user of this library has it do, as cases to be timed.

A case is one call (or one training step) through the public entry points of
`paper_2411_11547_amd`: the forward through a plan, the plan-free forward, the
Viterbi score, the adjoint, a training step through the autograd function, and
the forward over batches in host memory.  The shape of a case (batches, read
and haplotype lengths) follows from the case alone, the bases and qualities
from the seed.  Regions look like those of the benchmark's batches: haplotypes
are mutated copies of a reference, reads come from the haplotypes with
sequencing errors, base qualities are Illumina-like.
"""
import math

import numpy as np
import torch

from paper_2411_11547_amd import binding
from paper_2411_11547_amd.autograd import pairhmm_log10_likelihood
from paper_2411_11547_amd.workloads import Problem

MAX_PLAN_FREE_PAIRS = 65536


def _case(kind, regions, reads, haps, read_len, hap_len, shape=1, err=0.01, snp=0.004, n_rate=0.0, low_q=0.0, **more):
    """reads, haps, read_len, hap_len: (lowest, highest); counts and haplotype
    lengths are spread over their logarithm from region to region, read
    lengths evenly from read to read.  err: substitutions per read base;
    snp: per haplotype base; n_rate: N per read base; low_q: share of reads
    whose base qualities are all 2..10."""
    return dict(kind=kind, regions=regions, reads_lo=reads[0], reads_hi=reads[1], haps_lo=haps[0], haps_hi=haps[1],
                read_lo=read_len[0], read_hi=read_len[1], hap_lo=hap_len[0], hap_hi=hap_len[1], shape=shape, err=err,
                snp=snp, n_rate=n_rate, low_q=low_q, **more)


def listed():
    return [
        # one small active region of a variant caller, scored through a plan
        # and buffers that the caller keeps: latency and launches
        dict(name="forward 32 pairs", **_case("forward", 1, (8, 8), (4, 4), (100, 100), (150, 150))),
        # the batch of equal-length reads that throughput is quoted on
        dict(name="forward uniform", **_case("forward", 1000, (64, 64), (8, 8), (150, 150), (300, 300))),
        # a chromosome's worth of active regions, mixed lengths: the headline batch
        dict(name="forward mixed", **_case("forward", 2000, (10, 1000), (1, 28), (50, 250), (100, 1000))),
        # divergent haplotypes and low-quality reads: most pairs leave the
        # FP32 range and are done again in FP64
        dict(name="forward divergent", **_case("forward", 20000, (1, 1), (1, 1), (250, 250), (1000, 5000), snp=0.10,
                                               n_rate=0.02, low_q=0.3)),
        # long reads (HiFi-like) against local haplotypes: windows of rows
        dict(name="forward long reads", **_case("forward", 24, (1, 2), (1, 2), (1100, 8000), (3000, 9000), err=0.002)),
        # a serving loop that meets each region once and cannot allocate:
        # a single region, then a request of several
        dict(name="plan-free one region", **_case("plan-free", 1, (60, 60), (6, 6), (50, 250), (350, 350))),
        dict(name="plan-free 48 regions", **_case("plan-free", 48, (10, 200), (1, 16), (50, 250), (100, 1000))),
        # best-path scores of a mixed batch
        dict(name="viterbi mixed", **_case("viterbi", 300, (10, 1000), (1, 28), (50, 250), (100, 1000))),
        # parameter gradients of independent pairs
        dict(name="backward pairs", **_case("backward", 10000, (1, 1), (1, 1), (150, 150), (200, 600))),
        # parameter gradients of regions, every read shared by its region's haplotypes
        dict(name="backward regions", **_case("backward", 60, (10, 300), (1, 16), (50, 250), (100, 1000))),
        # one step of learning the parameters: log-likelihoods and the
        # gradient with explicit parameters, through autograd
        dict(name="training step", **_case("train", 16, (10, 60), (2, 8), (60, 300), (200, 600))),
        # batches that live in host memory, scored as they stream through
        dict(name="host batches", **_case("host", 600, (10, 1000), (1, 28), (50, 250), (100, 1000))),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# kind: most cells, most pairs of a drawn case
_LIMITS = {"forward": (1.2e11, 4e6), "viterbi": (6e10, 2e6), "backward": (6e9, 2e5), "train": (3e9, 1e5),
           "plan-free": (2e10, MAX_PLAN_FREE_PAIRS), "host": (6e10, 2e6)}


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "divergent", "long", "plan-free", "plan-free", "viterbi",
                       "backward", "backward", "train", "host"])
    shape = rng.randrange(1, 1 << 30)
    if kind == "divergent":
        n = _log_int(rng, 500, 3000)
        m = rng.randint(60, 300)
        case = _case("forward", _log_int(rng, 50, 20000), (1, 1), (1, 1), (m, m), (n, min(5000, 5 * n)), shape=shape,
                     snp=rng.uniform(0.05, 0.15), n_rate=0.02, low_q=0.3)
    elif kind == "long":
        m = _log_int(rng, 1100, 4000)
        n = _log_int(rng, 2000, 4500)
        case = _case("forward", rng.randint(1, 24), (1, 2), (1, 2), (m, 2 * m), (n, 2 * n), shape=shape, err=0.002)
    else:
        top = {"forward": 2000, "viterbi": 400, "host": 800, "plan-free": 64, "train": 40, "backward": 100}[kind]
        low = {"host": 20}.get(kind, 1)
        m = _log_int(rng, 30, 240)
        n = _log_int(rng, 100, 500)
        most = {"backward": 310, "train": 310}.get(kind, 600)
        case = _case(kind, _log_int(rng, low, top), (rng.randint(1, 20), rng.randint(20, 400)),
                     (rng.randint(1, 3), rng.randint(3, 24)), (m, min(most, m + rng.randint(0, 200))),
                     (n, n * rng.randint(1, 3)), shape=shape, n_rate=rng.choice([0.0, 0.002]))
    cells, pairs = _LIMITS[case["kind"]]
    while True:
        s = _Shape(case)
        if s.cells <= cells and s.pairs <= pairs:
            return case
        case["regions"] = max(1, case["regions"] * 2 // 3)
        if case["regions"] == 1:
            case["reads_hi"] = max(case["reads_lo"], case["reads_hi"] * 2 // 3)


class _Shape:
    """Counts and lengths of a case, and the batch structure they make."""

    def __init__(self, c):
        rng = np.random.default_rng([c["shape"], c["regions"]])

        def spread(lo, hi, size):
            return np.rint(np.exp(rng.uniform(math.log(lo), math.log(hi), size))).astype(np.int64)

        Q = c["regions"]
        self.R, self.H = spread(c["reads_lo"], c["reads_hi"], Q), spread(c["haps_lo"], c["haps_hi"], Q)
        self.ref = spread(c["hap_lo"], c["hap_hi"], Q)
        self.hap_region = np.repeat(np.arange(Q), self.H)
        # half of the haplotypes carry an insertion or a deletion of 1..5 bases
        nh = len(self.hap_region)
        self.indel = np.where(rng.random(nh) < 0.5, 0, rng.choice([-5, -4, -3, -2, -1, 1, 2, 3, 4, 5], nh))
        if c["hap_lo"] == c["hap_hi"]:  # haplotypes cut to one length
            self.n = self.ref[self.hap_region]
        else:
            self.n = self.ref[self.hap_region] + self.indel
        self.read_region = np.repeat(np.arange(Q), self.R)
        self.m = np.minimum(rng.integers(c["read_lo"], c["read_hi"] + 1, len(self.read_region)),
                            (self.ref - 6)[self.read_region])
        self.rb, self.hb = np.concatenate([[0], np.cumsum(self.R)]), np.concatenate([[0], np.cumsum(self.H)])
        self.ro, self.ho = np.concatenate([[0], np.cumsum(self.m)]), np.concatenate([[0], np.cumsum(self.n)])
        self.pairs = int((self.R * self.H).sum())
        self.cells = int((np.add.reduceat(self.m, self.rb[:-1]) * np.add.reduceat(self.n, self.hb[:-1])).sum())


def _ranges(lengths, dev):
    """(owner, position within the owner) of every element of back-to-back runs."""
    lengths = torch.as_tensor(lengths, device=dev)
    owner = torch.repeat_interleave(torch.arange(len(lengths), device=dev), lengths)
    first = torch.cumsum(lengths, 0) - lengths
    return owner, torch.arange(len(owner), device=dev) - first[owner]


def _data(c, s, seed):
    """Bases and qualities of a case from the seed: device uint8 tensors."""
    dev = "cuda"
    g = torch.Generator(device=dev).manual_seed(int(seed) * 1000003 + c["shape"])

    def ints(lo, hi, size):
        return torch.randint(lo, hi, (size,), generator=g, device=dev, dtype=torch.int64)

    def rand(size):
        return torch.rand(size, generator=g, device=dev)

    def at(a):
        return torch.as_tensor(a, device=dev)

    ref_len = s.ref + 16
    ref_off = at(np.concatenate([[0], np.cumsum(ref_len)])[:-1])
    ref = ints(0, 4, int(ref_len.sum()))
    owner, j = _ranges(s.n, dev)
    where = (rand(len(s.n)) * at(s.n)).long()
    src = j - torch.where(j > where[owner], at(s.indel)[owner], 0)
    src = src.clamp(min=0) + ref_off[at(s.hap_region)[owner]]
    hap = ref[src]
    hap = torch.where(rand(len(hap)) < c["snp"], (hap + ints(1, 4, len(hap))) % 4, hap)
    # every read from a place in a haplotype of its region
    region = at(s.read_region)
    pick = at(s.hb[:-1])[region] + (rand(len(s.m)) * at(s.H)[region]).long()
    start = at(s.ho[:-1])[pick] + (rand(len(s.m)) * (at(s.n)[pick] - at(s.m) + 1)).long()
    owner, k = _ranges(s.m, dev)
    base = hap[start[owner] + k]
    if c["snp"] > 0.02:  # divergent haplotypes: the reads come from the reference
        at_ref = ref_off[region] + (start - at(s.ho[:-1])[pick])
        base = ref[(at_ref[owner] + k).clamp(max=len(ref) - 1)]
    size = len(base)
    base = torch.where(rand(size) < c["err"], (base + ints(1, 4, size)) % 4, base)
    base = torch.where(rand(size) < c["n_rate"], 4, base)
    u, high = rand(size), ints(13, 41, size)
    bq = torch.where(u < 0.05, ints(2, 13, size), torch.where(u < 0.65, 37, torch.where(high >= 37, high + 1, high)))
    bq = torch.where((rand(len(s.m)) < c["low_q"])[owner], ints(2, 11, size), bq)
    b = {"read_bases": base, "base_qual": bq, "ins_qual": ints(40, 46, size), "del_qual": ints(40, 46, size),
         "gcp_qual": torch.full((size,), 10, device=dev), "hap_bases": hap}
    return {f: v.to(torch.uint8) for f, v in b.items()}


def _problem(c, s, d):
    h = {f: v.cpu().numpy() for f, v in d.items()}
    return Problem(s.rb, s.hb, s.ro, h["read_bases"], h["base_qual"], h["ins_qual"], h["del_qual"], h["gcp_qual"],
                   s.ho, h["hap_bases"])


def _upstream(s, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 17)
    return torch.rand(s.pairs, generator=g, device="cuda", dtype=torch.float64) + 0.5


def _log10_params(d):
    """{alpha, beta, delta, eps, zeta, lam_match, lam_mismatch} of every read
    base from its qualities, as float32 log10 values."""
    p = {f: torch.pow(10.0, -v.double() / 10) for f, v in d.items() if f.endswith("qual")}
    Q, de, ze, ep = p["base_qual"], p["ins_qual"], p["del_qual"], p["gcp_qual"]
    return torch.log10(torch.stack([1 - de - ze, 1 - ep, de, ep, ze, 1 - Q, Q / 3], 1)).float()


def prepare(case, seed):
    s = _Shape(case)
    d = _data(case, s, seed)
    problem = _problem(case, s, d)
    kind = case["kind"]
    if kind == "host":
        return {"kind": kind, "pipe": binding.Pipeline(problem)}
    state = {"kind": kind, "problem": problem, "dev": binding.DeviceProblem(problem)}
    if kind in ("forward", "viterbi", "plan-free"):
        state["out"] = torch.empty(s.pairs, dtype=torch.float64, device="cuda")
        state["status"] = torch.empty(s.pairs, dtype=torch.uint8, device="cuda")
    if kind != "plan-free":
        # autograd's buffers change from step to step, and a plan's graphs hold
        # for one set of buffers: a training loop launches directly
        state["plan"] = binding.Plan(problem, keep_checkpoints=kind in ("backward", "train"), use_graph=kind != "train")
    if kind in ("backward", "train"):
        state["up"] = _upstream(s, seed)
    if kind == "backward":
        state["grad"] = torch.empty((int(s.ro[-1]), 7), dtype=torch.float32, device="cuda")
    if kind == "train":
        state["params"] = _log10_params(d).requires_grad_(True)
    return state


def run(state):
    kind = state["kind"]
    if kind == "forward":
        return state["plan"].forward(state["dev"], out=state["out"], status=state["status"])
    if kind == "viterbi":
        return state["plan"].viterbi(state["dev"], out=state["out"], status=state["status"])
    if kind == "plan-free":
        return binding.forward_noalloc(state["problem"], state["dev"], out=state["out"], status=state["status"])
    if kind == "backward":
        return state["plan"].backward(state["dev"], state["up"], grad_params=state["grad"])
    if kind == "host":
        return state["pipe"].forward()
    params = state["params"]
    params.grad = None
    ll = pairhmm_log10_likelihood(params, state["plan"], state["dev"])
    (ll * state["up"]).sum().backward()
    return {"log10L": ll.detach(), "grad": params.grad}


def work(case):
    """Inputs read once, results written once; 11 operations per cell of the
    forward (8 of the Viterbi score), 37 with the adjoint (11 more for the
    reverse recurrences, 15 for the parameters' sums)."""
    s = _Shape(case)
    kind = case["kind"]
    bases = int(s.ro[-1])
    size = 5 * bases + int(s.ho[-1]) + 8 * (len(s.m) + len(s.n)) + 9 * s.pairs
    if kind == "backward":
        size += 28 * bases - s.pairs
    if kind == "train":
        size += (2 * 28 - 4) * bases + 8 * s.pairs
    per_cell = {"viterbi": 8, "backward": 37, "train": 37}.get(kind, 11)
    return {"bytes": size, "flops": per_cell * s.cells}


# ---------------------------------------------------------------------------
# the same results by the definition, in 64 bits
# ---------------------------------------------------------------------------
_SCALE = 2.0 ** 900


def _sweep(theta, read, hap, m, n, best):
    """L (best: the best path's probability) times _SCALE of a block of pairs,
    diagonal by diagonal: theta [pairs, rows, 7], read [pairs, rows] codes,
    hap [pairs, columns] codes with 5 past the end."""
    al, be, de, ep, ze, lm, lx = theta.unbind(2)
    dev, (B, rows), cols = read.device, read.shape, hap.shape[1]
    pad = torch.full((B, rows), 5, dtype=hap.dtype, device=dev)
    rev = torch.cat([pad, hap.flip(1), pad], 1)
    zero = torch.zeros((B, 1), dtype=torch.float64, device=dev)
    start = (_SCALE / n.double())[:, None]
    plus = torch.maximum if best else torch.add

    def above(x, edge):
        return torch.cat([edge, x[:, :-1]], 1)

    def blank():
        return torch.zeros((B, rows), dtype=torch.float64, device=dev)

    M1 = I1 = D1 = blank()  # diagonal d - 1, rows 1..rows
    M2 = I2 = D2 = blank()  # diagonal d - 2
    total = zero[:, 0]
    last = (m - 1)[:, None]
    wild = read == 4
    for d in range(2, rows + cols + 1):
        # row i meets column d - i: reversed haplotype from column d - 1 on
        code = rev[:, rows + cols - d + 1:rows + cols - d + 1 + rows]
        lam = torch.where(wild | (code == 4) | (code == read), lm, lx) * (code != 5)
        edge = start if d <= cols + 1 else zero
        ID = be * plus(above(I2, zero), above(D2, edge))
        M = lam * plus(al * above(M2, zero), ID)
        I = plus(de * above(M1, zero), ep * above(I1, zero))
        D = plus(ze * M1, ep * D1)
        end = plus(M, I).gather(1, last)[:, 0]
        total = plus(total, end)
        M2, I2, D2, M1, I1, D1 = M1, I1, D1, M, I, D
    return total


def _blocks(s, most):
    """Pairs in blocks of similar size, so that little is padded."""
    r = np.concatenate([np.repeat(np.arange(a, b), h) for a, b, h in zip(s.rb[:-1], s.rb[1:], s.H)])
    h = np.concatenate([np.tile(np.arange(a, b), k) for a, b, k in zip(s.hb[:-1], s.hb[1:], s.R)])
    order = np.lexsort((s.n[h], s.m[r] // 16))
    k = 0
    while k < len(order):
        e = min(len(order), k + max(1, int(most(int(s.m[r[order[k]]]) + 16, int(s.n[h].max())))))
        at = order[k:e]
        yield at, r[at], h[at]
        k = e


def exact(case, seed):
    s = _Shape(case)
    kind = case["kind"]
    grad = kind in ("backward", "train")
    if s.cells > (6e9 if grad else 4e10) or s.pairs > 1500000:
        return None  # tens of seconds
    d = _data(case, s, seed)
    dev = "cuda"
    if kind == "train":
        theta = torch.pow(10.0, _log10_params(d).double())
    else:
        p = {f: torch.pow(10.0, -v.double() / 10) for f, v in d.items() if f.endswith("qual")}
        Q, de, ze, ep = p["base_qual"], p["ins_qual"], p["del_qual"], p["gcp_qual"]
        theta = torch.stack([1 - de - ze, 1 - ep, de, ep, ze, 1 - Q, Q / 3], 1)
    t10 = torch.log10(theta)
    ro, ho, m_all, n_all = (torch.as_tensor(x, device=dev) for x in (s.ro, s.ho, s.m, s.n))
    out = torch.zeros(s.pairs, dtype=torch.float64, device=dev)
    sums = torch.zeros_like(theta) if grad else None
    up = _upstream(s, seed) if grad else None
    if grad:
        def most(m, n):
            return 2.5e10 / (m * (m + n) * 200.0)
    else:
        def most(m, n):
            return 6e7 / m
    for at, r, h in _blocks(s, most):
        at, r, h = (torch.as_tensor(x, device=dev) for x in (at, r, h))
        m, n = m_all[r], n_all[h]
        i = torch.arange(int(m.max()), device=dev)[None]
        pos = ro[r][:, None] + torch.minimum(i, (m - 1)[:, None])
        j = torch.arange(int(n.max()), device=dev)[None]
        hap = d["hap_bases"][ho[h][:, None] + torch.minimum(j, (n - 1)[:, None])]
        hap = torch.where(j < n[:, None], hap, 5)
        read = d["read_bases"][pos]
        if grad:
            leaf = t10[pos].requires_grad_(True)
            val = torch.log10(_sweep(torch.pow(10.0, leaf), read, hap, m, n, False)) - math.log10(_SCALE)
            (val * up[at]).sum().backward()
            part = torch.where((i < m[:, None])[:, :, None], leaf.grad, 0.0)
            sums.index_add_(0, pos.reshape(-1), part.reshape(-1, 7))
            out[at] = val.detach()
            del leaf, val, part
        else:
            out[at] = torch.log10(_sweep(theta[pos], read, hap, m, n, kind == "viterbi")) - math.log10(_SCALE)
    if kind == "backward":
        return sums
    if kind == "train":
        return {"log10L": out, "grad": sums}
    if kind == "host":
        return out.cpu().numpy(), None
    return out, None
