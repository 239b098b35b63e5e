"""The linear layers' walk over their tiles, on the CPU: every tile is taken once, and no load of any work-group reads past the
rows of x or of w, whether or not the scalar offset takes part in the hardware's range check."""
import pytest

from tests import linear_rule as rule

_FAULT = {1: "a tile is taken twice", 2: "a tile is missed", 3: "loads of the wrong tile or step", 4: "a live row is out of range",
          5: "a load reads past the end", 6: "work without rows"}


def follow(nj, mt, rows, N, K, cap=None):
    fault = rule.lib().linear_walk_check(nj, mt, max(rows, 1) if cap is None else cap, rows, N, K)
    assert fault == 0, (_FAULT.get(fault, fault), nj, mt, rows, N, K, cap)


def test_shapes_are_the_library_s():
    assert [(nj, mt) for nj, mt, _ in rule.shapes()] == rule.SHAPES


@pytest.mark.parametrize("nj,mt", rule.SHAPES)
def test_every_load_stays_inside_its_operand(nj, mt):
    stages = {s[:2]: s[2] for s in rule.shapes()}[nj, mt]
    tm, tn = 32 * mt, 32 * nj
    for K in (64, 128, 64 * (stages - 1), 64 * (stages + 2), 768):
        for rows in (1, tm - 1, tm, tm + 1, 3 * tm + 17, 9 * tm + 1):
            for feature_tiles in (1, 3, 7, 13):
                follow(nj, mt, rows, tn * feature_tiles, K)
        follow(nj, mt, 40 * tm + 5, tn * 20, K)                 # several tiles per work-group
        follow(nj, mt, tm + 3, tn * 2, K, cap=50 * tm)          # far fewer rows than the capacity
    follow(nj, mt, 2 * tm + 1, tn, 1 << 22)                     # the widest rows there are
    follow(nj, mt, 0, tn * 3, 768, cap=tm)


@pytest.mark.parametrize("nj,mt", rule.SHAPES)
def test_a_negative_device_row_count_is_no_work(nj, mt):
    """The number of tiles of such a count must not wrap round to a positive one."""
    for rows in (-1, -32 * mt, -32 * mt - 1, -(1 << 30), -(1 << 31) + 1, -(1 << 31)):
        for n_tiles in (1, 24, 33, 48, 63, 64, 96, 128, 512):
            follow(nj, mt, rows, 32 * nj * n_tiles, 64, cap=300)
