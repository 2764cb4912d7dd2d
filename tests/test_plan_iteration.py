"""Which units the planner gives the Gram-space iteration when a plan holds
units on both sides of its flop rule (L >= 1.25 S), and how many launches that
leaves (CPU)."""

import pytest

from paper_2510_16981_amd import muonbp as mb

WIDE = (512, 2048, 1, 1)      # L = 4 S: Gram-space by flops
SQUARE = (512, 512, 1, 1)     # L = S: as printed by flops
NARROW = (96, 512, 1, 1)      # S below the Gram-space floor: always as printed
LARGE = (4096, 14336, 1, 1), (4096, 4096, 1, 1)

# K = 5: 15 launches as printed, 17 in Gram space (segments of 3 and 2), 23 of
# both kinds.
CASES = [
    ([WIDE], 1, 17),
    ([SQUARE], 0, 15),
    ([WIDE, SQUARE], 2, 17),             # small: six launches outweigh the products' rate
    ([WIDE, SQUARE, NARROW], 1, 23),     # the floor keeps both kinds, so nothing to save
    ([WIDE, NARROW], 1, 23),
    (list(LARGE), 1, 23),                # large: the flop rule stands
]


@pytest.mark.parametrize("mats,units,launches", CASES)
def test_one_kind_of_iteration_on_small_plans(mats, units, launches):
    info = mb.describe_plan(mats, True)
    assert (info.gram_units, info.gemm_launches) == (units, launches)


def test_options_still_decide():
    mats = [WIDE, SQUARE]
    for mode, units in ((1, 0), (2, 2)):
        assert mb.describe_plan(mats, True, mb.options_default(gram_iteration=mode)).gram_units == units
    # A forced tile shape keeps the flop rule; one iteration has no Gram-space form.
    assert mb.describe_plan(mats, True, mb.options_default(tile_policy=8)).gram_units == 1
    assert mb.describe_plan(mats, True, mb.options_default(ns_steps=1)).gram_units == 0


def test_other_coefficients_keep_the_flop_rule():
    """Beyond the paper's quintic, only what ran in Gram space before does."""
    steep = dict(coeffs=[(3.4445, -4.7750, 2.0315), (2.0, -1.5, 0.5)])
    odd = (129, 1000, 1, 1)
    assert mb.describe_plan([WIDE, SQUARE], True, mb.options_default(**steep)).gram_units == 1
    assert mb.describe_plan([odd], True).gram_units == 1
    assert mb.describe_plan([odd], True, mb.options_default(**steep)).gram_units == 0
    assert mb.describe_plan([WIDE, odd], True, mb.options_default(a=3.0)).gram_units == 0
    assert mb.describe_plan([odd], True, mb.options_default(coeffs=[(2.0, -1.5, 0.5)] * 3)).gram_units == 1
