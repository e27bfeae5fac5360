"""The variant timer does not time two names of one launch: its choice holds for
a whole power of two of sizes, and which of two equal times is the smaller would
decide what runs at the others.  On the CPU, from the launch plans."""

import ctypes

import pytest

from tests.test_tune_gate import L, names, plan  # noqa: F401  (L: the fixture)


def timed(L, kind, n, per_cu=4):
    return {v for v in names(L, kind) if plan(L, kind, v, n, per_cu)[1]}


def default(L, kind, n):
    L.nbody_selected_variant.argtypes = [ctypes.c_int, ctypes.c_int64]
    return names(L, kind)[L.nbody_selected_variant(kind, n)]


# sizes at which the default variant runs the row-group kernel, and every
# variant that does so there
@pytest.mark.parametrize("kind,n,rows", [
    (0, 4097, ("fwd_row", "fwd_sym_w1_k2")), (0, 5000, ("fwd_row", "fwd_sym_w1_k2")),
    (0, 9000, ("fwd_row", "fwd_sym_w1_k2")), (0, 10499, ("fwd_row", "fwd_sym_w1_k2")),
    (1, 4096, ("bwd_row", "bwd_sym_s2")), (1, 6199, ("bwd_row", "bwd_sym_s2"))])
def test_row_groups_once(L, kind, n, rows):  # noqa: F811
    assert {v for v in timed(L, kind, n) if v.startswith(rows)} == {default(L, kind, n)}


@pytest.mark.parametrize("kind,n,rows", [(0, 4095, ("fwd_row",)), (0, 1000, ("fwd_row",)),
                                         (1, 4095, ("bwd_row",)), (1, 1000, ("bwd_row",))])
def test_row_variants_below(L, kind, n, rows):  # noqa: F811
    got = timed(L, kind, n)
    assert {v for v in names(L, kind) if v.startswith(rows)} <= got
    assert n < 4000 or "bwd_sym_s2_k2_r8" not in got


# one tile per wave: the variants whose plan holds it launch the default's grid
@pytest.mark.parametrize("kind,n,per_cu,same", [
    (0, 20000, 16, {"fwd_sym_w1_k4_r8", "fwd_sym_w1_k4_o1"}),
    (0, 45000, 4, {"fwd_sym_w4_k4_r8"}), (0, 45000, 16, {"fwd_sym_w1_k4_r8", "fwd_sym_w4_k4_r8"}),
    (0, 12000, 28, {"fwd_sym_w1_k2_r8", "fwd_sym_w1_k2_o1"}),
    (1, 8000, 8, {"bwd_sym_s2_k2_r8", "bwd_sym_s2_k2_r16", "bwd_sym_w1_k2_r8", "bwd_sym_w1_k2_r16"}),
    (1, 20000, 8, {"bwd_sym_s2_k2_r8", "bwd_sym_s2_k2_r16", "bwd_sym_w1_k2_r8", "bwd_sym_w1_k2_r16"})])
def test_one_tile_plans_once(L, kind, n, per_cu, same):  # noqa: F811
    assert timed(L, kind, n, per_cu) & same == {default(L, kind, n)}


@pytest.mark.parametrize("per_cu", [4])
def test_default_plan_holds_a_tile_per_wave_over_its_range(L, per_cu):  # noqa: F811
    # 40,000 bodies to the end of the range: the slots of the 4-wave blocks' plan
    # against those of blocks of 256, four tiles to a workgroup
    def fits(n):
        M = -(-n // 256)
        need = (4 * (M // 2 + 1) + 3) // 4 + M // 2
        return need <= plan(L, 0, "fwd_sym_w4_k4_r8", n, per_cu)[0] // (16 * n)

    assert default(L, 0, 40000) == default(L, 0, 49999) == "fwd_sym_w4_k4_r8"
    assert all(fits(n) for n in range(40000, 49153, 31)) and fits(49152)
    # the timer's view of the same line: another name of that launch, then not
    assert plan(L, 0, "fwd_sym_w1_k4_r8", 49152, 16)[1] == 0
    assert plan(L, 0, "fwd_sym_w1_k4_r8", 49153, 16)[1] == 1


@pytest.mark.parametrize("kind,variant,n", [(0, "fwd_sym_w1_k2_o1", 4096), (0, "fwd_sym_w1_k2_r8", 10499),
                                            (1, "bwd_sym_s2_k2_r8", 4000), (1, "bwd_sym_s2_k2_r16", 6199)])
def test_row_groups_take_no_workspace(L, kind, variant, n, monkeypatch):  # noqa: F811
    assert plan(L, kind, variant, n, 8)[0] == 0
    monkeypatch.setenv("NBODY_SYM_WORKSPACE", str(16 * n * 4))
    assert plan(L, kind, variant, n, 8)[0] == 0
    monkeypatch.setenv("NBODY_SYM_WORKSPACE", str(16 * n * 4 - 1))  # as the plan's own limit
    assert plan(L, kind, variant, n, 8)[0] == -1
