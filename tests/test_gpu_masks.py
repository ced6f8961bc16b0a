"""Preprocessing from per-state action masks (at most 64 actions): pi_pre, the
action counts and the action ranks against the oracle's Algorithm 4, and the
rounds that take over when two masks collide."""
import os

import numpy as np
import pytest

import oracle
from paper_2105_11788_amd import gen
from test_gpu_refine import _preprocessed, assert_parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2105_11788_amd import bisim
    return bisim


# (states, transitions, actions, initial blocks): one lane, partial waves, one
# action (Algorithm 2's initial partition is kept), all 64 mask bits, more
# states than one pass of the grid's workgroups, no transitions
@pytest.mark.parametrize("n,m,K,init", [
    (1, 0, 1, 0), (1, 3, 64, 1), (63, 200, 1, 0), (65, 300, 2, 3), (257, 0, 5, 4),
    (1000, 5000, 64, 0), (1000, 30000, 64, 7), (20000, 30000, 33, 300), (300000, 400000, 3, 2)])
def test_masks_match_the_rounds(B, n, m, K, init):
    L = gen.random_lts(n, m, K, seed=n + m + K, init_blocks=init)
    pre = oracle.preprocess(L.n, L.K, L.src, L.lab, L.dst, L.init)
    for collide in (False, True):
        method, pb, nm = _preprocessed(B, L, collide=collide)
        assert method == 0
        assert np.array_equal(pb, pre["pre_block"]) and np.array_equal(nm, pre["nr_marks"])
    if n <= 1000:  # the whole run also checks the action ranks
        assert_parity(B, L)
        os.environ["BISIM_ONEPASS_COLLIDE"] = "1"
        try:
            assert_parity(B, L)
        finally:
            os.environ.pop("BISIM_ONEPASS_COLLIDE", None)
