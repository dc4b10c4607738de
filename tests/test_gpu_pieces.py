"""Chains swept in pieces (a part of a larger batch keeps the larger plan's chain
length but takes shorter tiles): the host-input pipeline with its default subsets
gives the bits of a resident plan over the whole batch."""
import numpy as np
import pytest

from gpu_util import binding, gpu_forward, oracle, say, wl

pytestmark = pytest.mark.gpu


def test_default_subsets_equal_resident_plan():
    """2e10 cells, one default subset, cut into halves: the whole takes chains of
    2,048 or 4,096 columns, a half's own choice is shorter."""
    rng = np.random.default_rng(6)
    base = wl.config2(seed=6, regions=40)
    # the same regions over and over: 2e10 cells without their generation
    k = int(2e10 / base.total_cells) + 1
    rep = lambda a: np.tile(a, k)
    off = lambda o: np.concatenate([[0], np.cumsum(np.tile(np.diff(o), k))])
    prob = wl.Problem(off(base.batch_read_begin), off(base.batch_hap_begin), off(base.read_offset), rep(base.read_bases),
                      rep(base.base_qual), rep(base.ins_qual), rep(base.del_qual), rep(base.gcp_qual),
                      off(base.hap_offset), rep(base.hap_bases))
    pipe = binding.Pipeline(prob)
    say(f"{prob.num_pairs} pairs, {pipe.num_cells:.3g} cells, {pipe.num_subsets} subsets")
    assert pipe.num_subsets == 2 or (pipe.num_subsets == 3 and pipe.num_cells > 2.9e10)
    got, st = pipe.forward()
    pipe.close()
    ref, rst = gpu_forward(prob)
    assert np.array_equal(st, rst)
    assert np.array_equal(got, ref)
    # every copy of a region has the same scores
    assert np.abs(got.reshape(k, -1) - got[:base.num_pairs]).max() <= 1e-5
    pairs = np.sort(rng.choice(base.num_pairs, 50, replace=False))
    assert np.abs(got[pairs] - oracle.forward(base, pairs=pairs)).max() <= 1e-3
