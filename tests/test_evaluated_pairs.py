"""The pair counts that throughput figures rest on, at sizes where a pair-once
variant runs row groups."""

import pytest

from paper_0904_3659_amd import metrics
from tests.test_tune_gate import L, plan  # noqa: F401  (L: the fixture)


@pytest.mark.parametrize("variant,n,once", [
    ("fwd_sym_w1_k2_o1", 4095, True), ("fwd_sym_w1_k2_o1", 4096, False), ("fwd_sym_w1_k2_r8", 10499, False),
    ("fwd_sym_w1_k2_r8", 10500, True), ("fwd_sym_w1_k4_r8", 6001, True), ("fwd_row_k2", 6001, False),
    ("bwd_sym_s2_k2_r8", 3999, True), ("bwd_sym_s2_k2_r8", 6199, False), ("bwd_sym_s2_k2_r8", 6200, True),
    ("bwd_sym_w1_k2_r8", 5000, True), ("fwd_b256_k1_u8", 50000, False)])
def test_single_systems(variant, n, once):
    p = metrics.pairs(n)
    assert metrics.is_pair_once(variant, n) is once
    assert metrics.evaluated_pairs(p, variant) == (p // 2 if once else p)


def test_ensembles_and_no_size():
    assert metrics.evaluated_pairs(4999 * 5000, "bat_symd_w1_k4") == 4999 * 2500
    assert metrics.evaluated_pairs(0, "fwd_sym_w1_k2_o1") == 0
    assert metrics.is_pair_once("fwd_sym_w1_k2_o1") and not metrics.is_pair_once("bat_b64_u8")


def test_bands_are_the_library_s(L):  # noqa: F811
    # the timer passes one of two names of the row-group launch by: at the edges
    # of the bands, and only inside them
    timed = lambda kind, v, n: plan(L, kind, v, n, 8)[1]
    lo, hi = metrics.ROW_GROUPS["fwd_sym_w1_k2_"]
    assert [timed(0, "fwd_sym_w1_k2_r8", n) for n in (lo - 1, lo)] == [1, 0]
    assert [timed(0, "fwd_row_k1", n) for n in (hi - 1, hi)] == [0, 1]
    lo, hi = metrics.ROW_GROUPS["bwd_sym_s2_k2_"]
    assert [timed(1, "bwd_sym_s2_k2_r16", n) for n in (lo - 1, lo)] == [1, 0]
    assert [timed(1, "bwd_row_k1", n) for n in (hi - 1, hi)] == [0, 1]
