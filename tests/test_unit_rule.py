"""Host check of the rule that gives attention calls of few or short units workgroups of their own (`csrc/unit_rule.h`, plain host code), over
units, table widths, row bounds and cache types on both sides of its lines."""
import itertools

import pytest

from tests.helpers import unit_rule

CUS = 256
UNITS = list(range(1, 34)) + [40, 42, 43, 48, 63, 64, 65, 96, 127, 128, 129, 192, 255, 256, 257, 400, 511, 512, 513, 1280, 1536]
TILES = list(range(1, 140)) + [159, 160, 161, 255, 256, 257, 320, 511, 512, 513, 1023, 1024, 1025, 5000]
ROWS = [1, 16, 17, 32, 33, 48, 49, 64, 80]


@pytest.mark.parametrize("kv8", [False, True])
def test_shares_fit_the_chip_and_their_slots(kv8):
    for units, tiles, rows in itertools.product(UNITS, TILES, ROWS):
        splits, team = unit_rule(units, tiles, rows, kv8, CUS)
        what = (units, tiles, rows, splits, team)
        if splits == 0:
            assert tiles > 24, what                                # short units always take the path
            continue
        assert team in (4, 8) and 1 <= splits <= 16, what
        assert splits == 1 or units * splits <= CUS, what          # all shares at once on the chip, and a partial slot for each
        assert -(-tiles // splits) <= (80 if splits == 1 else 64), what


@pytest.mark.parametrize("kv8", [False, True])
def test_wide_tables_are_left_to_the_streaming_kernels(kv8):
    for units, rows in itertools.product(UNITS, ROWS):
        assert unit_rule(units, 1025, rows, kv8, CUS)[0] == 0


@pytest.mark.parametrize("kv8", [False, True])
def test_no_long_walk_by_one_workgroup_beside_idle_ones(kv8):
    """With compute units to spare a unit of more than 24 tiles (e4m3: 32) is shared out: one workgroup alone takes up to 40 % longer than the
    streaming kernels do with a plan that is there already."""
    for units, tiles, rows in itertools.product(range(1, 33), range(33, 49), ROWS):
        splits, team = unit_rule(units, tiles, rows, kv8, CUS)
        assert splits == -(-tiles // 8) and team == 4, (units, tiles, rows)


def test_long_shares_of_many_rows_are_refused():
    """From four row blocks on a share is bound by its instructions, which the streaming kernels spread over the chip."""
    for rows, kv8 in itertools.product((49, 64, 80), (False, True)):
        assert unit_rule(64, 160, rows, kv8, CUS)[0] == 0 and unit_rule(32, 320, rows, kv8, CUS)[0] == 0
        assert unit_rule(96, 65, rows, kv8, CUS)[0] == 0
    assert unit_rule(64, 160, 48, False, CUS)[0] == 4 and unit_rule(64, 80, 80, False, CUS)[0] == 0
