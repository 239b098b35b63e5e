"""The linear layers' walk over their tiles, on the CPU: every tile is taken once, and no load of any work-group reads past the
rows of x or of w, whether or not the scalar offset takes part in the hardware's range check."""
import pytest

from tests import linear_rule as rule

_FAULT = {1: "a tile is taken twice", 2: "a tile is missed", 3: "loads of the wrong tile or step", 4: "a live row is out of range",
          5: "a load reads past the end", 6: "work without rows"}


def follow(shape, rows, N, K, cap=None):
    fault = rule.lib().linear_walk_check(*shape, max(rows, 1) if cap is None else cap, rows, N, K)
    assert fault == 0, (_FAULT.get(fault, fault), shape, rows, N, K, cap)


def test_shapes_are_the_library_s():
    """Of the list that the kernels come from and of the rule's table."""
    assert list(rule.stages()) == rule.SHAPES
    assert rule.table() == rule.SHAPES


@pytest.mark.parametrize("shape", rule.SHAPES)
def test_every_load_stays_inside_its_operand(shape):
    stages = rule.stages()[shape]
    tm, tn = 32 * shape[1], 32 * shape[0]
    for K in (64, 128, 64 * (stages - 1), 64 * (stages + 2), 768):
        for rows in (1, tm - 1, tm, tm + 1, 3 * tm + 17, 9 * tm + 1):
            for feature_tiles in (1, 3, 7, 13):
                follow(shape, rows, tn * feature_tiles, K)
        follow(shape, 40 * tm + 5, tn * 20, K)                 # several tiles per work-group
        follow(shape, tm + 3, tn * 2, K, cap=50 * tm)          # far fewer rows than the capacity
    follow(shape, 2 * tm + 1, tn, 1 << 22)                     # the widest rows there are
    follow(shape, 0, tn * 3, 768, cap=tm)


def test_wide_outputs():
    """Tiles whose rows together have 2^32 bytes or more of output are not taken, all smaller ones are open; and with more panels
    than the walk passes one by one, every tile is still taken once."""
    taken = set()
    for N in (1 << 22, (1 << 22) + 768, (1 << 23) - 768, 1 << 23, 1 << 24, 1 << 25, (1 << 26) - 64):
        for rows in (1, 33, 100, 500, 2000):
            for K in (64, 1024):
                (nj, mt, per_cu), _ = rule.pick(rows, rows, N, K, "none")
                assert 32 * mt * N * 2 < 1 << 32, (N, rows, K, mt)
                taken.add((N, mt))
    assert max(mt for N, mt in taken if 1 << 22 < N < 1 << 23) == 8
    assert max(mt for N, mt in taken if N == 1 << 23) in (4, 5, 6, 7)
    assert rule.pick(500, 500, 1 << 26, 1024, "none")[0] == (2, 1, 1)
    for shape in rule.SHAPES:
        follow(shape, 32 * shape[1] + 1, 32 * shape[0] * 1999, 64)


@pytest.mark.parametrize("shape", rule.SHAPES)
def test_a_negative_device_row_count_is_no_work(shape):
    """The number of tiles of such a count must not wrap round to a positive one."""
    nj, mt, _ = shape
    for rows in (-1, -32 * mt, -32 * mt - 1, -(1 << 30), -(1 << 31) + 1, -(1 << 31)):
        for n_tiles in (1, 24, 33, 48, 63, 64, 96, 128, 512):
            follow(shape, rows, 32 * nj * n_tiles, 64, cap=300)
